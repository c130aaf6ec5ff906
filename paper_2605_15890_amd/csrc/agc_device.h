// Device-side building blocks of the gfx950 kernels: Philox4x32-10, DPP wave reductions and
// the two encode drivers (cyclic-band register ring, generic CSR gather).
//
// Thread geometry shared by the scale pass and the encode+quantize+pack pass: a wave covers
// one block of 256 consecutive coordinates, lane l owning the float4 at coordinates 4l..4l+3
// (the max-abs scale pass may give a wave two neighbouring blocks at once); a workgroup is
// four waves unless a kernel says otherwise.  Every lane walks over all workers for its
// coordinates, so the coded gradient f_i = sum_j a_ij g_j (Sec. II-A) only ever lives in
// registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "agc_kernels.h"

namespace agc {

constexpr int kMaxWorkers = 256;
constexpr int kWave = 64;
constexpr int kBlockCoords = 256;  // coordinates per wave pass
constexpr int kWavesPerWg = 4;
constexpr int kWgThreads = kWave * kWavesPerWg;
constexpr int kSegBlocks = 4;   // blocks per segment of the norm's summation tree
constexpr int kGroupSegs = 64;  // segments per group, groups per supergroup
constexpr int kMaxBand = 8;     // largest replication factor served by the register ring

// ---------------------------------------------------------------------------------------
// Philox4x32 with ten rounds (Salmon et al., SC'11).  Round: the two 32x32->64 products of
// counter words 0 and 2 with fixed odd multipliers; high halves are mixed with words 1 and 3
// and the round key; the key advances by Weyl constants.  On gfx950 the wide product is one
// full-rate v_mad_u64_u32 and the two mixes are one three-input xor each, so a block costs
// about 40 vector instructions.
// ---------------------------------------------------------------------------------------
// a ^ b ^ c in one instruction (gfx950's three-input bitwise op; truth table 0x96 = parity)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
#ifdef AGC_ABLATE_PHILOX
    constexpr int kRounds = 1;
#else
    constexpr int kRounds = 10;
#endif
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t pa = (uint64_t)0xD2511F53u * c0;
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(pb >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(pa >> 32), c3, k1);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// ---------------------------------------------------------------------------------------
// wave-wide reductions on the DPP cross-lane network (no LDS traffic)
// ---------------------------------------------------------------------------------------
constexpr int kDppQuadSwap1 = 0xB1;     // quad_perm [1,0,3,2]: partner l ^ 1
constexpr int kDppQuadSwap2 = 0x4E;     // quad_perm [2,3,0,1]: partner l ^ 2
constexpr int kDppHalfMirror = 0x141;   // l -> 7 - l within 8 lanes: a partner in the other quad
constexpr int kDppRowMirror = 0x140;    // l -> 15 - l within 16 lanes: a partner in the other half

constexpr int kDppQuadReverse = 0x1B;   // quad_perm [3,2,1,0]: l -> l ^ 3
constexpr int kDppRowRor4 = 0x124;      // rotation of 16 lanes by four
constexpr int kDppRowRor8 = 0x128;      // rotation of 16 lanes by eight: l -> l ^ 8

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// maximum over the wave of non-negative floats, returned as a wave-uniform bit pattern
// (non-negative floats order like their bit patterns)
__device__ __forceinline__ uint32_t wave_max_nonneg_bits(float x)
{
    uint32_t v = __float_as_uint(x);
    v = max(v, dpp_u32<kDppQuadSwap1>(v));
    v = max(v, dpp_u32<kDppQuadSwap2>(v));
    v = max(v, dpp_u32<kDppHalfMirror>(v));
    v = max(v, dpp_u32<kDppRowMirror>(v));  // every 16-lane row now holds its maximum
    const uint32_t r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const uint32_t r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    // the four row maxima are wave-uniform: combine them on the scalar unit (left to itself the
    // compiler moves them back into vector registers for a three-operand maximum)
    uint32_t a, b, m;
    asm("s_max_u32 %0, %1, %2" : "=s"(a) : "s"(r0), "s"(r1) : "scc");
    asm("s_max_u32 %0, %1, %2" : "=s"(b) : "s"(r2), "s"(r3) : "scc");
    asm("s_max_u32 %0, %1, %2" : "=s"(m) : "s"(a), "s"(b) : "scc");
    return m;
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_u32<CTRL>((uint32_t)b), hi = dpp_u32<CTRL>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Exchange-add over lanes at distances 1,2,4,8,16,32 (second level of the norm's tree),
// result wave-uniform.  After the steps at distance 1 and 2 every quad is uniform, so the
// mirror partners used for distances 4 and 8 hold exactly the value of lane l^4 and l^8; after
// distance 8 every 16-lane row is uniform and the last two steps are (r0+r1)+(r2+r3) on the
// four row values, which is what lanes of rows 0 and 1 compute in the exchange (rows 2 and 3
// compute the commuted, identical sum).
__device__ __forceinline__ double wave_butterfly_add(double v)
{
    v = v + dpp_f64<kDppQuadSwap1>(v);
    v = v + dpp_f64<kDppQuadSwap2>(v);
    v = v + dpp_f64<kDppHalfMirror>(v);
    v = v + dpp_f64<kDppRowMirror>(v);
    const double r0 = readlane_f64(v, 0), r1 = readlane_f64(v, 16);
    const double r2 = readlane_f64(v, 32), r3 = readlane_f64(v, 48);
    const double a = r0 + r1, b = r2 + r3;
    return a + b;
}

// Exchanges that keep several workers' values apart in the lanes' low bits.  After the first one a lane goes on with one
// of two workers (lanes with `second` with b); the sums of every worker are the same pairs as in wave_butterfly_add.
template <int CTRL>
__device__ __forceinline__ double exchange_pair(double a, double b, bool second)
{
    const double keep = second ? b : a, send = second ? a : b;
    return keep + dpp_f64<CTRL>(send);
}
__device__ __forceinline__ double exchange_quads(double v)  // distances 4 and 8
{
    v = v + dpp_f64<kDppQuadReverse>(dpp_f64<kDppHalfMirror>(v));  // l ^ 7 ^ 3
    return v + dpp_f64<kDppRowRor8>(v);
}
__device__ __forceinline__ double exchange_halves(double v)  // distances 16 and 32
{
    uint32_t lo = (uint32_t)(uint64_t)__double_as_longlong(v), hi = (uint32_t)((uint64_t)__double_as_longlong(v) >> 32);
    const auto l16 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h16 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __longlong_as_double((long long)(((uint64_t)h16[0] << 32) | l16[0])) + __longlong_as_double((long long)(((uint64_t)h16[1] << 32) | l16[1]));
    lo = (uint32_t)(uint64_t)__double_as_longlong(v);
    hi = (uint32_t)((uint64_t)__double_as_longlong(v) >> 32);
    const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __longlong_as_double((long long)(((uint64_t)h32[0] << 32) | l32[0])) + __longlong_as_double((long long)(((uint64_t)h32[1] << 32) | l32[1]));
}
// maxima over the wave of two workers' non-negative floats, the first's in the even lanes of the result, the second's in the
// odd ones (bit patterns; the maximum does not care for the order, so rotations by 4 and 8 will do)
__device__ __forceinline__ uint32_t pair_max_nonneg_bits(float a, float b, bool second)
{
    const uint32_t keep = __float_as_uint(second ? b : a), send = __float_as_uint(second ? a : b);
    uint32_t v = max(keep, dpp_u32<kDppQuadSwap1>(send));
    v = max(v, dpp_u32<kDppQuadSwap2>(v));
    v = max(v, dpp_u32<kDppRowRor4>(v));
    v = max(v, dpp_u32<kDppRowRor8>(v));
    const auto r16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max((uint32_t)r16[0], (uint32_t)r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return max((uint32_t)r32[0], (uint32_t)r32[1]);
}

// ---------------------------------------------------------------------------------------
// loads of one lane's float4
// ---------------------------------------------------------------------------------------
struct LaneCoords {
    int lane4;         // which float4 of the block the lane loads (clamped into the vector for lanes past d)
    uint32_t byte_off; // 16 * lane4: the lane's offset inside the block, as the 32-bit part of the address
    int nvalid;        // how many of the lane's four coordinates are < d (0..4)
    bool wave_ragged;  // wave-uniform: some lane of this wave has nvalid < 4
};

// base: first coordinate of the wave's block (wave-uniform, < d)
__device__ __forceinline__ LaneCoords lane_coords(int64_t base, int lane, int64_t d)
{
    LaneCoords lc;
    const int64_t left = d - base - 4 * lane;
    lc.nvalid = left >= 4 ? 4 : (left > 0 ? (int)left : 0);
    const int64_t last4 = (d - 1 - base) >> 2;  // last float4 of the block that holds a coordinate < d
    lc.lane4 = last4 < lane ? (int)last4 : lane;
    lc.byte_off = 16u * (uint32_t)lc.lane4;
    lc.wave_ragged = __any(lc.nvalid < 4) != 0;
    return lc;
}

// f with zeros for the lane's coordinates >= d
__device__ __forceinline__ float4 valid_coords(const float4& f, int nvalid)
{
    return make_float4(nvalid > 0 ? f.x : 0.f, nvalid > 1 ? f.y : 0.f, nvalid > 2 ? f.z : 0.f, nvalid > 3 ? f.w : 0.f);
}

// An epilogue behind a driver for the block that the vector ends in: it sees zeros for the coordinates >= d.  For
// epilogues that count them (Epi::kWantsZeros).
template <class Epi>
struct DropPast {
    static constexpr bool kStoresPerWorker = Epi::kStoresPerWorker;
    static constexpr int kPrefetchRows = Epi::kPrefetchRows;
    Epi& epi;
    int nvalid;
    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f) { epi.template worker<EVEN>(i, valid_coords(f, nvalid)); }
    __device__ __forceinline__ void worker_any(int i, const float4& f) { epi.worker_any(i, valid_coords(f, nvalid)); }
};

// `row` points at the block's first coordinate inside one row of G and is wave-uniform, so
// the load is a scalar base plus a 32-bit lane offset.  Every lane loads (lanes past d re-read
// the last float4, whose coordinates >= d are the row's padding), so there is no per-lane predicate; what comes of
// them is dropped behind the driver (DropPast).
// STREAM: the element is used once per pass (register-ring driver); a non-temporal load keeps it
// from displacing anything in the caches (measured: 9 % off the scale pass).  The gather driver
// re-reads rows and wants them cached.
template <bool STREAM>
__device__ __forceinline__ float4 load_row4(const float* __restrict__ row, const LaneCoords& lc)
{
    // scalar row pointer + zero-extended 32-bit lane offset: the form the hardware addresses
    // without any per-lane 64-bit arithmetic
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) char* global_bytes_t;
    typedef const __attribute__((address_space(1))) f32x4_t* global_f32x4_t;
    const global_f32x4_t src = (global_f32x4_t)((global_bytes_t)row + lc.byte_off);
#ifdef AGC_PLAIN_ROW_LOADS
    const f32x4_t t = *src;
#else
    const f32x4_t t = STREAM ? __builtin_nontemporal_load(src) : *src;
#endif
    return make_float4(t.x, t.y, t.z, t.w);
}

__device__ __forceinline__ float4 mul4(float a, const float4& g)
{
    return make_float4(a * g.x, a * g.y, a * g.z, a * g.w);
}
__device__ __forceinline__ float4 fma4(float a, const float4& g, const float4& c)
{
    return make_float4(fmaf(a, g.x, c.x), fmaf(a, g.y, c.y), fmaf(a, g.z, c.z), fmaf(a, g.w, c.w));
}

// What a lane holds of one row of G while it streams through a register ring: its float4 of one
// block (float4 itself), or its float4s of V neighbouring blocks (RowN<V>; the wave then covers
// 256 V consecutive coordinates and issues V loads per row, 1 KiB apart).  The multi-block form
// divides the number of row walks and of per-worker reductions by V; it is used where registers
// allow it (the max-abs scale pass).  All forms perform the same arithmetic on every coordinate.
template <int V>
struct RowN {
    float4 v[V];
};
typedef RowN<2> Row2;
template <int V>
__device__ __forceinline__ RowN<V> mul4(float c, const RowN<V>& g)
{
    RowN<V> r;
#pragma unroll
    for (int t = 0; t < V; ++t) r.v[t] = mul4(c, g.v[t]);
    return r;
}
template <int V>
__device__ __forceinline__ RowN<V> fma4(float c, const RowN<V>& g, const RowN<V>& f)
{
    RowN<V> r;
#pragma unroll
    for (int t = 0; t < V; ++t) r.v[t] = fma4(c, g.v[t], f.v[t]);
    return r;
}

// Row -> number of blocks
template <class Row>
struct RowBlocks {
    static constexpr int value = sizeof(Row) / sizeof(float4);
};

template <class Row>
__device__ __forceinline__ Row zero_row()
{
    Row r;
    float4* p = reinterpret_cast<float4*>(&r);
#pragma unroll
    for (int t = 0; t < RowBlocks<Row>::value; ++t) p[t] = make_float4(0.f, 0.f, 0.f, 0.f);
    return r;
}

// streaming load of a lane's part of a row whose blocks lie wholly inside the vector
template <class Row, bool STREAM = true>
__device__ __forceinline__ Row load_row(const float* __restrict__ row, const LaneCoords& lc)
{
    Row r;
    float4* p = reinterpret_cast<float4*>(&r);
#pragma unroll
    for (int t = 0; t < RowBlocks<Row>::value; ++t) p[t] = load_row4<STREAM>(row + t * kBlockCoords, lc);
    return r;
}

// ---------------------------------------------------------------------------------------
// Encode driver 1: cyclic band.  n == k, worker i stores columns (i+u) mod k, u = 0..S-1.
// Rows stream once through a ring of R = S + P row registers (P rows of prefetch); worker
// i is formed when row i+S-1 has arrived.  The first S-1 rows are kept in a register stash
// for the last S-1 workers, which wrap around, so every element of G is read exactly once.
// R is even so that the parity of the worker handled at each unrolled position is known at
// compile time (the quantizer shares one Philox block between workers 2q and 2q+1).  The
// epilogue is called for workers 0..n-1 in ascending order.
// ---------------------------------------------------------------------------------------
// PF = requested prefetch distance in rows (made one larger when S + PF would be odd)
template <int S, int PF>
struct RingShapeT {
    static constexpr int P = ((S + PF) & 1) ? PF + 1 : PF;
    static constexpr int R = S + P;
    static constexpr int NSTASH = S > 1 ? S - 1 : 1;
};
// The prefetch distance is a property of the epilogue (Epi::kPrefetchRows).  Quantize pass: two
// rows ahead (measured 2/3/4/6/8/10 rows: 1.393/1.402/1.400/1.411/1.419/1.414 ms on the metric
// workload, two rows also best on the smaller ones: deeper prefetch only costs registers, the
// pass does not wait for its loads).  One-block scale pass: two as well (Euclidean scale at the
// metric size: 0.972 ms against 0.983 ms with four).
#ifndef AGC_PREFETCH_ROWS
#define AGC_PREFETCH_ROWS 2
#endif
#ifndef AGC_SCALE_PREFETCH_ROWS
#define AGC_SCALE_PREFETCH_ROWS 2
#endif

// value select (the operands are read before the choice, so the choice is between registers)
__device__ __forceinline__ float4 sel4(bool c, const float4 a, const float4 b)
{
    return make_float4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}
template <int V>
__device__ __forceinline__ RowN<V> sel4(bool c, const RowN<V>& a, const RowN<V>& b)
{
    RowN<V> r;
#pragma unroll
    for (int t = 0; t < V; ++t) r.v[t] = sel4(c, a.v[t], b.v[t]);
    return r;
}

// stash helpers with compile-time indices (so the stash stays in registers)
template <int S, int PF, class Row, int... Us>
__device__ __forceinline__ Row stash_pick(const Row (&stash)[(RingShapeT<S, PF>::NSTASH)], int idx,
                                             std::integer_sequence<int, Us...>)
{
    Row v = stash[0];
    ((v = sel4(idx == Us + 1, stash[(Us + 1) < RingShapeT<S, PF>::NSTASH ? (Us + 1) : 0], v)), ...);
    return v;
}

template <int S, int PF, class Row, int r, int... Us>
__device__ __forceinline__ void stash_fill(Row (&stash)[(RingShapeT<S, PF>::NSTASH)],
                                           const Row (&ring)[(RingShapeT<S, PF>::R)],
                                           std::integer_sequence<int, Us...>)
{
    constexpr int R = RingShapeT<S, PF>::R;
    ((stash[Us] = ring[(r + R - (S - 1) + Us) % R]), ...);
}

// One row arrival.  STEADY rounds are straight-line code: every prefetch is issued (past the
// last row the last row is re-read, a cache hit whose value is never used), every worker index
// is valid and no wrapped row is involved, so the compiler can count outstanding loads exactly
// and let P of them stay in flight.  The first round and the last one or two (GENERAL) carry
// the conditions: workers that do not exist yet, the stash fill, the wrapped rows.
template <int S, int PF, class Row, int r, bool STEADY, class Epi>
__device__ __forceinline__ void ring_step(Row (&ring)[(RingShapeT<S, PF>::R)],
                                          Row (&stash)[(RingShapeT<S, PF>::NSTASH)],
                                          const float*& next_row, int64_t ldg, int k,
                                          const float* __restrict__ bval, const LaneCoords& lc,
                                          int j0, float (&coef)[S], Epi& epi)
{
    constexpr int P = RingShapeT<S, PF>::P;
    constexpr int R = RingShapeT<S, PF>::R;
    const int j = j0 + r;
    if (STEADY) {
        ring[(r + P) % R] = load_row<Row>(next_row, lc);
        next_row += (j + P + 1 < k) ? ldg : 0;  // stays on the last row once it is reached
    } else {
        if (j + P < k) {  // prefetch the row that arrives P steps from now
            ring[(r + P) % R] = load_row<Row>(next_row, lc);
            next_row += (j + P + 1 < k) ? ldg : 0;
        }
        if (S > 1 && j >= k && j < k + S - 1)  // arrivals k..k+S-2 are rows 0..S-2, kept in the stash
            ring[r] = stash_pick<S, PF, Row>(stash, j - k, std::make_integer_sequence<int, (S > 2 ? S - 2 : 0)>{});
    }
    const int i = j - (S - 1);
    if (STEADY || (i >= 0 && i < k)) {
        if (!STEADY && S > 1 && i == 0)
            stash_fill<S, PF, Row, r>(stash, ring, std::make_integer_sequence<int, (S > 1 ? S - 1 : 0)>{});
        // the worker's coefficients were requested one worker earlier (the scalar read is then
        // over by the time they are used); request the next worker's now
        float next[S];
        const float* bv = bval + (int64_t)(i + 1 < k ? i + 1 : i) * S;
#pragma unroll
        for (int u = 0; u < S; ++u) next[u] = bv[u];
        Row f = mul4(coef[0], ring[(r + R - (S - 1)) % R]);
#pragma unroll
        for (int u = 1; u < S; ++u) f = fma4(coef[u], ring[(r + R - (S - 1) + u) % R], f);
        epi.template worker<(((r + R - (S - 1)) & 1) == 0)>(i, f);
#pragma unroll
        for (int u = 0; u < S; ++u) coef[u] = next[u];
    }
}

template <int S, int PF, class Row, bool STEADY, class Epi, int... Rs>
__device__ __forceinline__ void ring_round(Row (&ring)[(RingShapeT<S, PF>::R)],
                                           Row (&stash)[(RingShapeT<S, PF>::NSTASH)],
                                           const float*& next_row, int64_t ldg, int k,
                                           const float* __restrict__ bval, const LaneCoords& lc,
                                           int j0, float (&coef)[S], Epi& epi, std::integer_sequence<int, Rs...>)
{
    (ring_step<S, PF, Row, Rs, STEADY>(ring, stash, next_row, ldg, k, bval, lc, j0, coef, epi), ...);
}

template <int S, int PF, class Row, class Epi>
__device__ __forceinline__ void encode_ring(const float* __restrict__ G, int64_t ldg, int k,
                                            const float* __restrict__ bval, const LaneCoords& lc,
                                            Epi& epi)
{
    constexpr int P = RingShapeT<S, PF>::P;
    constexpr int R = RingShapeT<S, PF>::R;
    static_assert(R % 2 == 0, "ring length must be even");
    constexpr auto seq = std::make_integer_sequence<int, R>{};
    const int steps = k + S - 1;  // row arrivals, the last S-1 being the wrapped rows
    Row ring[R];
    Row stash[(RingShapeT<S, PF>::NSTASH)];
    const float* next_row = G;  // G already points at the block's first coordinate in row 0
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = zero_row<Row>();
    stash[0] = zero_row<Row>();
#pragma unroll
    for (int r = 0; r < P; ++r) {
        if (r < k) {
            ring[r] = load_row<Row>(next_row, lc);
            next_row += (r + 1 < k) ? ldg : 0;
        }
    }
    float coef[S];  // coefficients of the worker that is formed next
#pragma unroll
    for (int u = 0; u < S; ++u) coef[u] = bval[u];
    int j0 = 0;
    ring_round<S, PF, Row, false>(ring, stash, next_row, ldg, k, bval, lc, j0, coef, epi, seq);
    for (j0 = R; j0 + R - 1 < k; j0 += R)
        ring_round<S, PF, Row, true>(ring, stash, next_row, ldg, k, bval, lc, j0, coef, epi, seq);
    for (; j0 < steps; j0 += R)
        ring_round<S, PF, Row, false>(ring, stash, next_row, ldg, k, bval, lc, j0, coef, epi, seq);
}

// ---------------------------------------------------------------------------------------
// Encode driver 2: any CSR code.  Each worker gathers its rows straight from memory; rows
// shared by neighbouring workers are served by the caches.
// ---------------------------------------------------------------------------------------
// Wave-uniform read of a small read-only table (code structure, per-worker records).  Tagging the
// address as constant memory keeps the read on the scalar path even in a kernel that also stores:
// otherwise the compiler must assume its own stores may have changed the table, reads it with a
// vector load and waits for every outstanding load and store.  Nothing writes these tables while
// a kernel that reads them runs.
template <class T>
__device__ __forceinline__ T load_uniform(const T* p)
{
    static_assert(sizeof(T) % 4 == 0, "whole dwords");
    constexpr int N = sizeof(T) / 4;
    const __attribute__((address_space(4))) uint32_t* q = (const __attribute__((address_space(4))) uint32_t*)p;
    uint32_t w[N];
#pragma unroll
    for (int t = 0; t < N; ++t) w[t] = q[t];
    T out;
    __builtin_memcpy(&out, w, sizeof(T));
    return out;
}

struct CsrView {
    const int* __restrict__ row_ptr;
    const int* __restrict__ col;
    const float* __restrict__ val;
    const WindowRec* __restrict__ win;  // monotone-interval codes: one record per row + sentinel
    const StreamRec* __restrict__ stream = nullptr;  // codes that stream_records takes: one record per entry + sentinel
    bool keep = false;                               // and G is small enough to be found in the caches again
};

__device__ __forceinline__ float4 encode_gather_one(const float* __restrict__ G, int64_t ldg,
                                                    const CsrView& B, int i, const LaneCoords& lc)
{
    const int e0 = B.row_ptr[i], e1 = B.row_ptr[i + 1];
    float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
    if (e0 < e1) {
        f = mul4(B.val[e0], load_row4<false>(G + (int64_t)B.col[e0] * ldg, lc));
        for (int e = e0 + 1; e < e1; ++e)
            f = fma4(B.val[e], load_row4<false>(G + (int64_t)B.col[e] * ldg, lc), f);
    }
    return f;
}

template <class Epi>
__device__ __forceinline__ void encode_gather(const float* __restrict__ G, int64_t ldg, int n,
                                              const CsrView& B, const LaneCoords& lc, Epi& epi)
{
    for (int i = 0; i < n; i += 2) {
        epi.template worker<true>(i, encode_gather_one(G, ldg, B, i, lc));
        if (i + 1 < n) epi.template worker<false>(i + 1, encode_gather_one(G, ldg, B, i + 1, lc));
    }
}

// ---------------------------------------------------------------------------------------
// Encode driver 3: monotone intervals.  Every worker stores a run of consecutive columns
// lo_i .. lo_i+len_i-1 (ascending, len_i <= W) and neither lo_i nor lo_i+len_i-1 decreases with i
// - the shape of the paper's sparse construction (Sec. III-A: contiguous allocation segments on
// the partition axis).  Rows stream once through the same register ring as the cyclic band; a
// worker is formed when row lo_i + W - 1 arrives, so that row lo_i + u sits at a ring position
// that is known at compile time; entries u >= len_i are skipped by wave-uniform branches (not
// multiplied by zero: the sum must have exactly the stored terms).  Several workers, or none, may
// be anchored at the same row.
// ---------------------------------------------------------------------------------------
// the part of a row's record the driver keeps in scalar registers
struct WindowCur {
    int lo, len;
    float val[8];
};

__device__ __forceinline__ WindowCur load_window_rec(const WindowRec* rec)
{
    struct Head { int lo, len; };
    struct Vals { float v[8]; };
    const Head h = load_uniform(reinterpret_cast<const Head*>(rec));
    const Vals v = load_uniform(reinterpret_cast<const Vals*>(rec->val));
    WindowCur c;
    c.lo = h.lo;
    c.len = h.len;
#pragma unroll
    for (int u = 0; u < 8; ++u) c.val[u] = v.v[u];
    return c;
}

template <int W, int PF, class Row, int r, bool STEADY, class Epi>
__device__ __forceinline__ void window_step(Row (&ring)[(RingShapeT<W, PF>::R)], const float*& next_row,
                                            int64_t ldg, int k, const CsrView& B, const LaneCoords& lc,
                                            int j0, int& i, WindowCur& cur, Epi& epi)
{
    constexpr int P = RingShapeT<W, PF>::P;
    constexpr int R = RingShapeT<W, PF>::R;
    const int j = j0 + r;
    if (STEADY || j + P < k) {  // prefetch the row that arrives P steps from now
        ring[(r + P) % R] = load_row<Row>(next_row, lc);
        next_row += (j + P + 1 < k) ? ldg : 0;
    }
    const int lo = j - (W - 1);
    while (cur.lo == lo) {  // the sentinel record ends the last run
        const WindowCur nxt = load_window_rec(B.win + i + 1);
        Row f = mul4(cur.val[0], ring[(r + R - (W - 1)) % R]);
#pragma unroll
        for (int u = 1; u < W; ++u)
            if (u < cur.len) f = fma4(cur.val[u], ring[(r + R - (W - 1) + u) % R], f);
        epi.worker_any(i, f);
        cur = nxt;
        ++i;
    }
}

template <int W, int PF, class Row, bool STEADY, class Epi, int... Rs>
__device__ __forceinline__ void window_round(Row (&ring)[(RingShapeT<W, PF>::R)], const float*& next_row,
                                             int64_t ldg, int k, const CsrView& B, const LaneCoords& lc,
                                             int j0, int& i, WindowCur& cur, Epi& epi,
                                             std::integer_sequence<int, Rs...>)
{
    (window_step<W, PF, Row, Rs, STEADY>(ring, next_row, ldg, k, B, lc, j0, i, cur, epi), ...);
}

template <int W, int PF, class Row, class Epi>
__device__ __forceinline__ void encode_window(const float* __restrict__ G, int64_t ldg, int k,
                                              const CsrView& B, const LaneCoords& lc, Epi& epi)
{
    constexpr int P = RingShapeT<W, PF>::P;
    constexpr int R = RingShapeT<W, PF>::R;
    constexpr auto seq = std::make_integer_sequence<int, R>{};
    Row ring[R];
    const float* next_row = G;
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = zero_row<Row>();
#pragma unroll
    for (int r = 0; r < P; ++r) {
        if (r < k) {
            ring[r] = load_row<Row>(next_row, lc);
            next_row += (r + 1 < k) ? ldg : 0;
        }
    }
    int i = 0;
    WindowCur cur = load_window_rec(B.win);
    int j0 = 0;
    const int steps = k + W - 1;  // the last worker may be anchored at row k-1
    for (; j0 + R - 1 + P < k; j0 += R)  // every prefetch of the round exists
        window_round<W, PF, Row, true>(ring, next_row, ldg, k, B, lc, j0, i, cur, epi, seq);
    for (; j0 < steps; j0 += R)
        window_round<W, PF, Row, false>(ring, next_row, ldg, k, B, lc, j0, i, cur, epi, seq);
}

// The same driver for epilogues that store inside the worker loop (the quantize pass).  Stores
// and loads share one outstanding-operation counter on this hardware, so behind a loop of unknown
// length the compiler can only wait for everything; a rolling prefetch would be drained at every
// row.  Here the rows arrive in batches of BT: while the BT row steps of one batch run, the next
// batch is in flight; it is waited for as a whole when its turn comes.  The ring holds the
// current batch, the next one and the up to W-1 older rows a worker may still need, rounded up to
// whole batches so that all positions stay compile-time.  The structure of worker i comes from
// its 64-byte record, read one worker ahead.
template <int W>
struct BatchShape {
    static constexpr int BT = 4;                                   // rows per batch
    static constexpr int R = ((2 * BT + W - 1 + BT - 1) / BT) * BT;  // current + next batch + W-1 older rows
    static constexpr int NB = R / BT;
};

template <int W, int H>
__device__ __forceinline__ void window_request(float4 (&ring)[BatchShape<W>::R], const float* __restrict__ G,
                                               int64_t ldg, int k, const LaneCoords& lc, int row0)
{
    constexpr int BT = BatchShape<W>::BT;
    if (row0 < k) {  // one straight run of loads; a batch that straddles the end repeats row k-1
#pragma unroll
        for (int r = 0; r < BT; ++r) {
            const int row = row0 + r < k ? row0 + r : k - 1;
            ring[H * BT + r] = load_row4<true>(G + (int64_t)row * ldg, lc);
        }
    }
}

template <int W, int H, class Epi>
__device__ __forceinline__ void window_batch(float4 (&ring)[BatchShape<W>::R], const float* __restrict__ G,
                                             int64_t ldg, int k, const CsrView& B, const LaneCoords& lc,
                                             int row0, int& i, WindowCur& cur, Epi& epi)
{
    constexpr int BT = BatchShape<W>::BT;
    constexpr int R = BatchShape<W>::R;
    constexpr int NB = BatchShape<W>::NB;
    // the batch requested one round ago has to be here now.  The empty asm makes its registers
    // plain values for the compiler from here on: without it every later row step waits for all
    // outstanding operations, the stores of the step before included.
#pragma unroll
    for (int r = 0; r < BT; ++r) {
        float4& x = ring[H * BT + r];
        asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
    }
    window_request<W, (H + 1) % NB>(ring, G, ldg, k, lc, row0 + BT);
#pragma unroll
    for (int r = 0; r < BT; ++r) {
        const int lo = row0 + r - (W - 1);
        while (cur.lo == lo) {  // the sentinel record ends the last run
            const WindowCur nxt = load_window_rec(B.win + i + 1);  // in flight during this worker
            float4 f = mul4(cur.val[0], ring[(H * BT + r + R - (W - 1)) % R]);
#pragma unroll
            for (int u = 1; u < W; ++u)
                if (u < cur.len) f = fma4(cur.val[u], ring[(H * BT + r + R - (W - 1) + u) % R], f);
            epi.worker_any(i, f);
            cur = nxt;
            ++i;
        }
    }
}

template <int W, int H, class Epi>
__device__ __forceinline__ void window_batches(float4 (&ring)[BatchShape<W>::R], const float* __restrict__ G,
                                               int64_t ldg, int k, const CsrView& B, const LaneCoords& lc,
                                               int row0, int steps, int& i, WindowCur& cur, Epi& epi)
{
    if constexpr (H < BatchShape<W>::NB) {
        if (row0 < steps) {
            window_batch<W, H>(ring, G, ldg, k, B, lc, row0, i, cur, epi);
            window_batches<W, H + 1>(ring, G, ldg, k, B, lc, row0 + BatchShape<W>::BT, steps, i, cur, epi);
        }
    }
}

template <int W, class Epi>
__device__ __forceinline__ void encode_window_batched(const float* __restrict__ G, int64_t ldg, int k,
                                                      const CsrView& B, const LaneCoords& lc, Epi& epi)
{
    constexpr int R = BatchShape<W>::R;
    float4 ring[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    int i = 0;
    WindowCur cur = load_window_rec(B.win);
    const int steps = k + W - 1;  // the last worker may be anchored at row k-1
    window_request<W, 0>(ring, G, ldg, k, lc, 0);
    for (int row0 = 0; row0 < steps; row0 += R)
        window_batches<W, 0>(ring, G, ldg, k, B, lc, row0, steps, i, cur, epi);
}

// ---------------------------------------------------------------------------------------
// Encode driver 4: monotone intervals of any length of which few are open at a time (a worker is open from its first column to
// its last).  Rows stream once; a row is added to every open worker's sum as it arrives and is then dropped, so the
// registers hold the sums of the open workers and the rows that are on their way.  A sum starts at -0, which
// makes the first fused multiply-add the rounded product, sign of zero included.  The lowest open worker is always the first
// to be complete.
// Up to 256 MB of G, which the memory-side cache holds, rows are loaded to be kept for the pass or step that follows, above
// that non-temporally.  Whole steps, us, the general driver (one row of one worker after the other) | this one kept | this one
// non-temporal: 10 workers and 30 partitions x 400 000 41.6 | 33.6 | 39.7, 900 000 49.2 | 43.3 | 45, 1.5 M 64.0 | 63.8 | 68,
// 2.5 M 126 | 109 | 110, 5.4 M 238-241 | 243 | 231;  24 and 70 x 5.4 M 539 | 555 | 512;  64 and 64 x 12.8 M 1607 | - | 1226.  Two
// rows ahead; with four, six and eight 10 x 5.4 M takes 244, 247 and 252: more waves fit with fewer registers.
// ---------------------------------------------------------------------------------------
constexpr int kStreamDriver = -64;  // the S of kernels with this driver
constexpr int64_t kKeepElements = (int64_t)1 << 26;
constexpr int kStreamAhead = 2;     // rows requested ahead

__device__ __forceinline__ float4 minus_zero(const float4&) { return make_float4(-0.f, -0.f, -0.f, -0.f); }
template <int V>
__device__ __forceinline__ RowN<V> minus_zero(const RowN<V>& r)
{
    RowN<V> z;
#pragma unroll
    for (int t = 0; t < V; ++t) z.v[t] = minus_zero(r.v[t]);
    return z;
}

template <class Row, bool STREAM, class Epi>
__device__ __forceinline__ void encode_stream_rows(const float* __restrict__ G, int64_t ldg, int k, const CsrView& B, const LaneCoords& lc,
                                                   Epi& epi)
{
    Row ring[kStreamAhead], open[kStreamSlots];
    const float* next_row = G;
    int left = k;  // rows not requested yet
#pragma unroll
    for (int r = 0; r < kStreamAhead; ++r) {
        ring[r] = load_row<Row, STREAM>(next_row, lc);  // past the last row the last row is read again
        left -= 1;
        next_row += left > 0 ? ldg : 0;
    }
#pragma unroll
    for (int t = 0; t < kStreamSlots; ++t) open[t] = minus_zero(ring[0]);
    const StreamRec* rec = B.stream;
    StreamRec cur = load_uniform(rec);
    int i = 0;
    for (int j0 = 0; j0 < k; j0 += kStreamAhead) {
#pragma unroll
        for (int r = 0; r < kStreamAhead; ++r) {
            while (cur.col == j0 + r) {
                const StreamRec nxt = load_uniform(++rec);
#pragma unroll
                for (int t = 0; t < kStreamSlots; ++t)
                    if (cur.slot == t) open[t] = fma4(cur.val, ring[r], open[t]);  // wave-uniform
                if (cur.last) {
                    epi.worker_any(i, open[0]);
                    ++i;
#pragma unroll
                    for (int t = 0; t + 1 < kStreamSlots; ++t) open[t] = open[t + 1];
                    open[kStreamSlots - 1] = minus_zero(ring[0]);
                }
                cur = nxt;
            }
            ring[r] = load_row<Row, STREAM>(next_row, lc);
            left -= 1;
            next_row += left > 0 ? ldg : 0;
        }
    }
}

template <class Row, class Epi>
__device__ __forceinline__ void encode_stream(const float* __restrict__ G, int64_t ldg, int k, const CsrView& B, const LaneCoords& lc,
                                              Epi& epi)
{
    if (B.keep) encode_stream_rows<Row, false>(G, ldg, k, B, lc, epi);
    else encode_stream_rows<Row, true>(G, ldg, k, B, lc, epi);
}

// ---------------------------------------------------------------------------------------
// The same drivers for a range of workers i0..i1-1 (i0 even, i0 < i1), for passes that give the waves of a
// workgroup a part of the workers each.  The cyclic band loads the rows that wrap around once more.
// ---------------------------------------------------------------------------------------
template <int S, int PF, int r, class Epi>
__device__ __forceinline__ void ring_part_step(float4 (&ring)[(RingShapeT<S, PF>::R)], const float* __restrict__ G,
                                               int64_t ldg, int k, const float* __restrict__ bval,
                                               const LaneCoords& lc, int j0, int i0, int m, int& row,
                                               float (&coef)[S], Epi& epi)
{
    constexpr int P = RingShapeT<S, PF>::P;
    constexpr int R = RingShapeT<S, PF>::R;
    const int j = j0 + r;
    if (j + P < m + S - 1) {
        ring[(r + P) % R] = load_row4<true>(G + (int64_t)row * ldg, lc);
        row = row + 1 < k ? row + 1 : 0;
    }
    const int t = j - (S - 1);
    if (t >= 0 && t < m) {
        const int i = i0 + t;
        float next[S];
        const float* bv = bval + (int64_t)(t + 1 < m ? i + 1 : i) * S;
#pragma unroll
        for (int u = 0; u < S; ++u) next[u] = bv[u];
        float4 f = mul4(coef[0], ring[(r + R - (S - 1)) % R]);
#pragma unroll
        for (int u = 1; u < S; ++u) f = fma4(coef[u], ring[(r + R - (S - 1) + u) % R], f);
        epi.template worker<(((r + R - (S - 1)) & 1) == 0)>(i, f);
#pragma unroll
        for (int u = 0; u < S; ++u) coef[u] = next[u];
    }
}

template <int S, int PF, class Epi, int... Rs>
__device__ __forceinline__ void ring_part_round(float4 (&ring)[(RingShapeT<S, PF>::R)], const float* __restrict__ G,
                                                int64_t ldg, int k, const float* __restrict__ bval,
                                                const LaneCoords& lc, int j0, int i0, int m, int& row,
                                                float (&coef)[S], Epi& epi, std::integer_sequence<int, Rs...>)
{
    (ring_part_step<S, PF, Rs>(ring, G, ldg, k, bval, lc, j0, i0, m, row, coef, epi), ...);
}

template <int S, int PF, class Epi>
__device__ __forceinline__ void encode_ring_part(const float* __restrict__ G, int64_t ldg, int k,
                                                 const float* __restrict__ bval, const LaneCoords& lc, int i0, int i1,
                                                 Epi& epi)
{
    constexpr int P = RingShapeT<S, PF>::P;
    constexpr int R = RingShapeT<S, PF>::R;
    const int m = i1 - i0;
    int row = i0;
    float4 ring[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int r = 0; r < P; ++r) {
        if (r < m + S - 1) {
            ring[r] = load_row4<true>(G + (int64_t)row * ldg, lc);
            row = row + 1 < k ? row + 1 : 0;
        }
    }
    float coef[S];
#pragma unroll
    for (int u = 0; u < S; ++u) coef[u] = bval[(int64_t)i0 * S + u];
    for (int j0 = 0; j0 < m + S - 1; j0 += R)
        ring_part_round<S, PF>(ring, G, ldg, k, bval, lc, j0, i0, m, row, coef, epi, std::make_integer_sequence<int, R>{});
}

template <int W, int PF, int r, class Epi>
__device__ __forceinline__ void window_part_step(float4 (&ring)[(RingShapeT<W, PF>::R)], const float* __restrict__ G,
                                                 int64_t ldg, int k, const CsrView& B, const LaneCoords& lc, int j0,
                                                 int i1, int& i, WindowCur& cur, Epi& epi)
{
    constexpr int P = RingShapeT<W, PF>::P;
    constexpr int R = RingShapeT<W, PF>::R;
    const int j = j0 + r;
    if (j + P < k) ring[(r + P) % R] = load_row4<true>(G + (int64_t)(j + P) * ldg, lc);
    const int lo = j - (W - 1);
    while (i < i1 && cur.lo == lo) {
        const WindowCur nxt = load_window_rec(B.win + i + 1);  // the sentinel record ends the table
        float4 f = mul4(cur.val[0], ring[(r + R - (W - 1)) % R]);
#pragma unroll
        for (int u = 1; u < W; ++u)
            if (u < cur.len) f = fma4(cur.val[u], ring[(r + R - (W - 1) + u) % R], f);
        epi.worker_any(i, f);
        cur = nxt;
        ++i;
    }
}

template <int W, int PF, class Epi, int... Rs>
__device__ __forceinline__ void window_part_round(float4 (&ring)[(RingShapeT<W, PF>::R)], const float* __restrict__ G,
                                                  int64_t ldg, int k, const CsrView& B, const LaneCoords& lc, int j0,
                                                  int i1, int& i, WindowCur& cur, Epi& epi,
                                                  std::integer_sequence<int, Rs...>)
{
    (window_part_step<W, PF, Rs>(ring, G, ldg, k, B, lc, j0, i1, i, cur, epi), ...);
}

// rows are counted from 0, ring positions from the first row the range needs
template <int W, int PF, class Epi>
__device__ __forceinline__ void encode_window_part(const float* __restrict__ G, int64_t ldg, int k, const CsrView& B,
                                                   const LaneCoords& lc, int i0, int i1, Epi& epi)
{
    constexpr int P = RingShapeT<W, PF>::P;
    constexpr int R = RingShapeT<W, PF>::R;
    int i = i0;
    WindowCur cur = load_window_rec(B.win + i);
    const int first = cur.lo / R * R;  // a whole number of rounds: row j sits at position j mod R
    float4 ring[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int r = 0; r < P; ++r)
        if (first + r < k) ring[r] = load_row4<true>(G + (int64_t)(first + r) * ldg, lc);
    for (int j0 = first; i < i1; j0 += R)  // every worker is met: its lo is at most k - 1
        window_part_round<W, PF>(ring, G, ldg, k, B, lc, j0, i1, i, cur, epi, std::make_integer_sequence<int, R>{});
}

template <class Epi>
__device__ __forceinline__ void encode_gather_part(const float* __restrict__ G, int64_t ldg, const CsrView& B,
                                                   const LaneCoords& lc, int i0, int i1, Epi& epi)
{
    for (int i = i0; i < i1; i += 2) {
        epi.template worker<true>(i, encode_gather_one(G, ldg, B, i, lc));
        if (i + 1 < i1) epi.template worker<false>(i + 1, encode_gather_one(G, ldg, B, i + 1, lc));
    }
}

// workers i0..i1-1 of one block; nothing if the range is empty
template <int S, class Epi>
__device__ __forceinline__ void encode_part_any(const float* __restrict__ G, int64_t ldg, int k, const CsrView& B,
                                                const LaneCoords& lc, int i0, int i1, Epi& epi)
{
    if constexpr (S > 0) encode_ring_part<S, Epi::kPrefetchRows>(G, ldg, k, B.val, lc, i0, i1, epi);
    else if constexpr (S < 0) encode_window_part<-S, Epi::kPrefetchRows>(G, ldg, k, B, lc, i0, i1, epi);
    else encode_gather_part(G, ldg, B, lc, i0, i1, epi);
}
template <int S, class Epi>
__device__ __forceinline__ void encode_block_part(const float* __restrict__ G, int64_t ldg, int k, const CsrView& B,
                                                  const LaneCoords& lc, int i0, int i1, Epi& epi)
{
    if (i0 >= i1) return;
    if (!Epi::kWantsZeros || !lc.wave_ragged) {
        encode_part_any<S>(G, ldg, k, B, lc, i0, i1, epi);
    } else {
        DropPast<Epi> drop{epi, lc.nvalid};
        encode_part_any<S>(G, ldg, k, B, lc, i0, i1, drop);
    }
}

// Short vectors: how many waves share the workers of a block (each takes a run of an even number of them).
constexpr int kParts = 4;
__host__ __device__ inline int part_size(int n) { return ((n + kParts - 1) / kParts + 1) / 2 * 2; }

// One block of 256 coordinates for all workers.  S > 0: cyclic band of width S; S < 0: monotone
// intervals of at most -S columns; S == 0: any code.  All give identical bits.  The block that straddles d takes
// the same driver as the others, in an instance of its own: with the test for it in the epilogues of all blocks, bucket-wise
// steps were 2-5 % slower.  It used to take the gather driver, n rows one after the other while the chip waited.
// Whole steps, gather | as now, us: 256 workers x 1 000 000, Euclidean 738 | 393, max-abs 618 | 389, one pass 485 | 291;
// 64 x 2 000 000 234 | 191;  128 x 5 400 001 1119 | 1047;  32 x 11 700 001 559 | 546;  16 x 300 001 23.8 | 21.4.
template <int S, class Epi>
__device__ __forceinline__ void encode_block_any(const float* __restrict__ G, int64_t ldg, int n, int k,
                                                 const CsrView& B, const LaneCoords& lc, Epi& epi)
{
    if constexpr (S == kStreamDriver) {
        encode_stream<float4>(G, ldg, k, B, lc, epi);
    } else if constexpr (S > 0) {
        encode_ring<S, Epi::kPrefetchRows, float4>(G, ldg, k, B.val, lc, epi);
    } else if constexpr (S < 0) {  // monotone intervals of at most -S columns
        if constexpr (Epi::kStoresPerWorker) encode_window_batched<-S>(G, ldg, k, B, lc, epi);
        else encode_window<-S, Epi::kPrefetchRows, float4>(G, ldg, k, B, lc, epi);
    } else {
        encode_gather(G, ldg, n, B, lc, epi);
    }
}
template <int S, class Epi>
__device__ __forceinline__ void encode_block(const float* __restrict__ G, int64_t ldg, int n, int k,
                                             const CsrView& B, const LaneCoords& lc, Epi& epi)
{
    if (!Epi::kWantsZeros || !lc.wave_ragged) {
        encode_block_any<S>(G, ldg, n, k, B, lc, epi);
    } else {
        DropPast<Epi> drop{epi, lc.nvalid};
        encode_block_any<S>(G, ldg, n, k, B, lc, drop);
    }
}

// epilogue for the largest-magnitude scale: exact and order-free
struct EpiMaxAbs {
    static constexpr bool kStoresPerWorker = false;
    static constexpr bool kWantsZeros = true;
    static constexpr int kPrefetchRows = AGC_SCALE_PREFETCH_ROWS;
    uint32_t* acc;  // this wave's LDS slice [n], bit patterns of non-negative floats
    int lane;
    static __device__ __forceinline__ float max_abs4(const float4& f)
    {
        return fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w)));
    }
    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f)
    {
        const uint32_t m = wave_max_nonneg_bits(max_abs4(f));
        if (lane == 0) acc[i] = m;
    }
    template <bool EVEN, int V>
    __device__ __forceinline__ void worker(int i, const RowN<V>& f)  // V blocks, one reduction
    {
        float a = max_abs4(f.v[0]);
#pragma unroll
        for (int t = 1; t < V; ++t) a = fmaxf(a, max_abs4(f.v[t]));
        const uint32_t m = wave_max_nonneg_bits(a);
        if (lane == 0) acc[i] = m;
    }
    template <class Row>
    __device__ __forceinline__ void worker_any(int i, const Row& f) { worker<true>(i, f); }
};

// multiplier of the grid positions: L_i * 2^16 / scale (2^15 / scale for a one-bit worker)
__device__ __forceinline__ float inv16_of(float scale, int bits)
{
    if (!(scale > 0.f)) return 0.f;
    const double num = bits >= 2 ? (double)((1 << (bits - 1)) - 1) * 65536.0 : 32768.0;
    const float q = (float)(num / (double)scale);
    return (q <= 3.402823466e+38f) ? q : 0.f;
}

}  // namespace agc
