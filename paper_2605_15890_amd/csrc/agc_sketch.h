// Worker side with ONE read of G, for scales of the whole vector.  The quantize pass needs every worker's scale, the scale
// needs the whole vector, and reading G twice is most of a step (64 workers x 25.6 M: 2 x 6.55 GB of 13.8).  But with a
// small magnitude against the scale nearly every coordinate ends at level 0 whatever the scale is exactly: for the
// Euclidean norm the levels sum to at most L * sqrt(d) of d coordinates.  So:
//   1. a sample of the vector, at places drawn anew for every step, gives a lower bound of every scale (launch_sketch_bounds);
//   2. k_sketch reads G once.  It forms the partial results of the scales and, with the bound in place of the scale,
//      the largest grid position a coordinate can have.  Where the draw lies above that, the level is 0 for every
//      scale from the bound upwards and only the sign is kept, one bit; the others are written down whole ("records": the
//      coded value, its draw, worker and place);
//   3. when the scales are known and none fell below its bound, k_resolve (agc_resolve.hip) makes the codes and the estimate
//      of signs and records, by the arithmetic of k_quantize, operation by operation;
//   4. groups of blocks with more records than there is room for, listed by k_resolve, or all if a bound did not hold, take
//      k_quantize.
// The results are those of the two-read form bit for bit, whatever the sample said.
//
// Measured, 64 workers x 25.6 M, three bits on average, Euclidean, interval code, whole step 2416 us with two reads (scale pass
// 984, quantize pass 1420), 1470 with one: sample and bounds 11 + 5, k_sketch 1210-1240, groups and finalize 12,
// k_resolve 224, the quantize pass that finds nothing left 7.  A step whose bounds do not hold pays for both forms (some 2670).
// Values that are not alike everywhere, two reads | one: rows of 16384 with the first 256 values 20 times the others, six bits,
// 64 x 25.6 M 2498 | 1744 (interval code 2560 | 1793), 50 x 5.4 M 433 | 351, 64 x 5.4 M three bits 529 | 350; sixty layers of magnitudes up
// to 1000 apart, eight bits, 64 x 25.6 M 2501 | 1915.  What stays slower: at 64 x 1 M the second pass takes 27 us for however few
// blocks, so a norm in a 64th of the vector or less, 112 | 119 (window of 8 132 | 148), and such rows, 113 | 115 (132 | 140), lose what
// alike values gain, 112 | 88 (132 | 104).
#pragma once

#include "agc_device.h"
#include "agc_kernels.h"
#include "agc_quantize.h"

namespace agc {

struct SketchArgs {
    int64_t ldg;
    int n, k;
    int64_t d;
    uint32_t key0, key1, step_lo, step_hi;
    const WindowRec* win;  // monotone-interval codes only
    const StreamRec* stream;  // codes that stream_records takes
    double* part_sq;       // Euclidean scale: [segment][worker]
    uint32_t* run_max;     // largest magnitude: [worker]
    SketchDev sk;
};

// The norm's exchange-add over the 64 lanes (wave_butterfly_add) for four workers at once: after the first exchange a
// lane goes on with one of two workers only, after the second with one of four, so that the later ones are shared.  Every
// worker's sums are the same pairs as alone.
__device__ __forceinline__ double sum_rows_of_four(double v)  // lane l: worker l & 3, sum of its quad -> of the wave
{
    return exchange_halves(exchange_quads(v));
}

// what the sketches of both kinds of scale have in common: draws and signs
struct SketchLane {
    static constexpr bool kStoresPerWorker = false;
    static constexpr bool kWantsZeros = true;
    static constexpr int kPrefetchRows = AGC_PREFETCH_ROWS;
    uint32_t key0, key1, step_lo, step_hi;
    uint32_t* plane;       // this wave's LDS slice, [worker][8]: 256 signs in the order of the coordinates
    int n;
    int lane;
    uint32_t ctr0;
    uint32_t keep0, keep1, keep2, keep3;  // the Philox block of a pair: two words of the even worker, two of the odd one
    uint32_t word;         // the lane's signs of the last eight workers, coordinate q of the newest at bit q

    __device__ __forceinline__ void draw(int i)
    {
        uint32_t o[4];
        philox4x32_10(ctr0, (uint32_t)i >> 1, step_lo, step_hi, key0, key1, o);
        keep0 = o[0];
        keep1 = o[1];
        keep2 = o[2];
        keep3 = o[3];
    }

    // Eight workers' nibbles of every lane -> per eight lanes eight dwords of one worker each, 32 coordinates in order: a
    // transpose in three exchanges.  The newest worker sits in nibble 0 and ends up in lane 0 of the eight.
    __device__ __forceinline__ void store_signs(int i)
    {
        uint32_t v = word << (4 * (7 - (i & 7)));
        const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
        uint32_t t = dpp_u32<kDppQuadSwap1>(v);
        t = __builtin_amdgcn_alignbit(t, t, b0 ? 4 : 28);
        const uint32_t m0 = b0 ? 0xF0F0F0F0u : 0x0F0F0F0Fu;
        v = (v & m0) | (t & ~m0);
        t = dpp_u32<kDppQuadSwap2>(v);
        t = __builtin_amdgcn_alignbit(t, t, b1 ? 8 : 24);
        const uint32_t m1 = b1 ? 0xFF00FF00u : 0x00FF00FFu;
        v = (v & m1) | (t & ~m1);
        t = dpp_u32<kDppQuadReverse>(dpp_u32<kDppHalfMirror>(v));
        t = __builtin_amdgcn_alignbit(t, t, 16);
        const uint32_t m2 = b2 ? 0xFFFF0000u : 0x0000FFFFu;
        v = (v & m2) | (t & ~m2);
        plane[(i >> 3) * kWave + (7 - (lane & 7)) * 8 + (lane >> 3)] = v;
    }
    __device__ __forceinline__ void keep_signs(int i, const float4& f)
    {
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.w), 31);
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.z), 31);
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.y), 31);
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.x), 31);
        if ((i & 7) == 7 || i == n - 1) store_signs(i);
    }
};

struct EpiSketch : SketchLane {
    const float* lo_mult;  // [n], scalar reads
    double* acc;           // this wave's LDS slices: [n]
    uint2* recs;           // [cap]
    int cap;
    int count;             // wave-uniform: records so far, with those that did not fit
    double sq, sq2;        // sums of squares that wait for the other worker of the pair, and for the other pair
    float pend;            // multiplier of the worker that comes next, requested one worker early

    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f)
    {
        if (EVEN) draw(i);
        take(i, f, EVEN ? keep0 : keep2, EVEN ? keep1 : keep3, EVEN);
    }
    __device__ __forceinline__ void worker_any(int i, const float4& f)
    {
        uint32_t wa = keep2, wb = keep3;
        if ((i & 1) == 0) {  // wave-uniform
            draw(i);
            wa = keep0;
            wb = keep1;
        }
        take(i, f, wa, wb, (i & 1) == 0);
    }
    // append a record of every lane of m: two counting instructions and one LDS store
    __device__ __forceinline__ void append(uint64_t m, bool here, float f, uint32_t u16, uint32_t place)
    {
        if (m == 0) return;
        const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)count));
        if (here && pos < (uint32_t)cap) recs[pos] = make_uint2(__float_as_uint(f), (u16 << 16) | place);
        count = __builtin_amdgcn_readfirstlane(count + __builtin_popcountll(m));
    }

    __device__ __forceinline__ void sum_of_four(int first, double v)
    {
        v = sum_rows_of_four(v);
        if (lane < 4 && first + lane < n) acc[first + lane] = v;
    }

    __device__ __forceinline__ void take(int i, const float4& f, uint32_t wa, uint32_t wb, bool even)
    {
        const float mult = pend;
        pend = load_uniform(lo_mult + (i + 1 < n ? i + 1 : i));
        {
            // squares are exact in binary64, so the fused sums round as the plain ones do
            const double x0 = f.x, x1 = f.y, x2 = f.z, x3 = f.w;
            const double q = fma(x0, x0, x1 * x1) + fma(x2, x2, x3 * x3);
            if (even) {
                sq = q;
            } else {
                const double pair = exchange_pair<kDppQuadSwap1>(sq, q, lane & 1);
                if ((i & 2) == 0) sq2 = pair;  // wave-uniform
                else sum_of_four(i - 3, exchange_pair<kDppQuadSwap2>(sq2, pair, lane & 2));
            }
        }
        keep_signs(i, f);
        // level 0 for every scale from the bound upwards: the grid position lies below the draw, so the true one,
        // which is no larger (product and quotient round monotonically), does too, and no tie can arise.  The draw is a
        // whole number, so the position need not be truncated for the comparison.
        const bool c0 = fabsf(f.x) * mult >= (float)(wa & 0xFFFFu), c1 = fabsf(f.y) * mult >= (float)(wa >> 16);
        const bool c2 = fabsf(f.z) * mult >= (float)(wb & 0xFFFFu), c3 = fabsf(f.w) * mult >= (float)(wb >> 16);
        const uint64_t m0 = __builtin_amdgcn_ballot_w64(c0), m1 = __builtin_amdgcn_ballot_w64(c1);
        const uint64_t m2 = __builtin_amdgcn_ballot_w64(c2), m3 = __builtin_amdgcn_ballot_w64(c3);
        if ((m0 | m1 | m2 | m3) != 0) {
            const uint32_t place = ((uint32_t)i << 8) | (4u * (uint32_t)lane);
            append(m0, c0, f.x, wa & 0xFFFFu, place);
            append(m1, c1, f.y, wa >> 16, place + 1u);
            append(m2, c2, f.z, wb & 0xFFFFu, place + 2u);
            append(m3, c3, f.w, wb >> 16, place + 3u);
        }
    }

    // after the last worker: the sums of an incomplete four
    __device__ __forceinline__ void finish()
    {
        const int left = n & 3;
        if (left == 0) return;
        double pair = sq2;  // left == 2: the one pair
        double other = 0.0;
        if (left != 2) other = exchange_pair<kDppQuadSwap1>(sq, 0.0, lane & 1);
        if (left == 1) {
            pair = other;
            other = 0.0;
        }
        sum_of_four(n - left, exchange_pair<kDppQuadSwap2>(pair, other, lane & 2));
    }
};

__device__ __forceinline__ void store_plane(const SketchArgs& a, int64_t block, const uint32_t* plane, int lane)
{
    asm volatile("" ::: "memory");  // the lanes read what others have written
    const u32x4_t* signs = reinterpret_cast<const u32x4_t*>(plane);
    const __amdgpu_buffer_rsrc_t out = uniform_buffer(a.sk.planes + block * (int64_t)(4 * a.sk.chunks * kWave), 32 * a.n);
    for (int p = lane; p < 2 * a.n; p += kWave)
        __builtin_amdgcn_raw_buffer_store_b128(signs[p], out, 16 * p, 0, kPayloadStorePolicy);
}

// What bounds it: stores among reads.  With the cyclic code the bare row walk takes 0.96 ms, the kernel without its stores
// 1.04, with the 205 MB of signs 1.21 (plain stores 1.235, non-temporal 1.218, written through as well 1.21); without
// the Philox rounds or the sums of squares it is not faster.  Three, four, five, six waves per SIMD: 1.47, 1.24, 1.215,
// 1.32 ms; four leave the most room for records.  Four workers' sums share their exchanges because vector
// instructions still count at that occupancy: 76 per worker and wave (the sums of each worker alone: 90).
//
// One wave per block of 256 coordinates, four blocks of a segment of the norm's tree per workgroup.
// LDS: [4][n] doubles, [4][4 * chunks][64] dwords of signs, [4][cap] records.
template <int S>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(S == 0 || S == kStreamDriver ? 1 : 4, S == 0 || S == kStreamDriver ? 8 : 4))) void k_sketch(
    const float* __restrict__ G, const int* __restrict__ row_ptr, const int* __restrict__ col,
    const float* __restrict__ val, const float* __restrict__ lo_mult, SketchArgs a)
{
    extern __shared__ __attribute__((aligned(16))) double lds_sketch[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t seg = blockIdx.x;
    const int64_t block = seg * kSegBlocks + wave;
    const int64_t base = block * (int64_t)kBlockCoords;
    double* acc = lds_sketch + wave * a.n;
    uint32_t* plane = reinterpret_cast<uint32_t*>(lds_sketch + kSegBlocks * a.n) + wave * (4 * a.sk.chunks * kWave);
    uint2* recs = reinterpret_cast<uint2*>(lds_sketch + kSegBlocks * a.n + kSegBlocks * 2 * a.sk.chunks * kWave) + wave * a.sk.cap;
    if (base < a.d) {
        const LaneCoords lc = lane_coords(base, lane, a.d);
        EpiSketch epi{{a.key0, a.key1, a.step_lo, a.step_hi, plane, a.n, lane, (uint32_t)((base + 4 * lane) >> 2)},
                      lo_mult, acc, recs, a.sk.cap, 0, 0.0, 0.0, load_uniform(lo_mult)};
        encode_block<S>(G + base, a.ldg, a.n, a.k, CsrView{row_ptr, col, val, a.win, a.stream, (int64_t)a.k * a.d <= kKeepElements}, lc, epi);
        epi.finish();
        // what this wave's lanes have left in LDS leaves in long runs, by the store policy of the payload
        store_plane(a, block, plane, lane);
        const int have = epi.count <= a.sk.cap ? epi.count : -1;
        const u32x4_t* from = reinterpret_cast<const u32x4_t*>(recs);
        const __amdgpu_buffer_rsrc_t list = uniform_buffer(a.sk.recs + block * (int64_t)a.sk.cap, 8 * a.sk.cap);
        for (int p = lane; 2 * p < have; p += kWave)
            __builtin_amdgcn_raw_buffer_store_b128(from[p], list, 16 * p, 0, kPayloadStorePolicy);
        if (lane == 0) a.sk.counts[block] = have;
    } else {
        for (int i = lane; i < a.n; i += kWave) acc[i] = 0.0;
        if (lane == 0) a.sk.counts[block] = 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < a.n; i += kWgThreads) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < kSegBlocks; ++w) sum = sum + lds_sketch[w * a.n + i];
        __builtin_nontemporal_store(sum, a.part_sq + seg * (int64_t)a.n + i);
    }
}

// Records of a wave wait in LDS, a ring of kRecRing, and leave by halves of it: a block's room is then a matter of memory, not of LDS.
// With all of a block's records in LDS (960 at 64 workers) a fifth of the groups of 64 workers x 25.6 M with heavy tails overflowed.
constexpr int kRecRing = 512;

struct EpiSketchMax : SketchLane {
    // send(): windows take their rows in batches, whose waits do not reach the records' stores.  Whole steps, 64 workers x 25.6 M, rows
    // one by one | in batches, us: runs of 4, heavy tails 2077 | 1731, layers 2396 (two reads 2356) | 2099;  runs of 8 2133 | 1856,
    // 2481 | 2237;  runs of 2, 32 x 35 M 1447 | 1183, 1736 (1600) | 1499.
    static constexpr bool kStoresPerWorker = true;
    const float* mult;     // this wave's LDS slices: [n] multipliers of the bounds
    uint32_t* acc;         // [n] largest magnitudes of the block
    uint2* ring;           // [kRecRing]
    uint2* recs;           // the block's records in memory
    int cap;               // a multiple of kRecRing / 2
    int count, gone;       // wave-uniform: records so far; of these, in memory
    float top;             // the largest magnitude that waits for the other worker of the pair
    float pend;            // multiplier of the worker that comes next, requested one worker early

    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f)
    {
        if (EVEN) draw(i);
        take(i, f, EVEN ? keep0 : keep2, EVEN ? keep1 : keep3, EVEN);
    }
    __device__ __forceinline__ void worker_any(int i, const float4& f)
    {
        uint32_t wa = keep2, wb = keep3;
        if ((i & 1) == 0) {  // wave-uniform
            draw(i);
            wa = keep0;
            wb = keep1;
        }
        take(i, f, wa, wb, (i & 1) == 0);
    }
    __device__ __forceinline__ void append(uint64_t m, bool here, float f, uint32_t u16, uint32_t place)
    {
        if (m == 0) return;
        const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)count));
        if (here) ring[pos & (kRecRing - 1)] = make_uint2(__float_as_uint(f), (u16 << 16) | place);
        count = __builtin_amdgcn_readfirstlane(count + __builtin_popcountll(m));
    }
    __device__ __forceinline__ void send(int pieces)  // from `gone` on, pieces of two records
    {
        asm volatile("" ::: "memory");  // the lanes read what others have written
        const u32x4_t* from = reinterpret_cast<const u32x4_t*>(ring + (gone & (kRecRing - 1)));
        const __amdgpu_buffer_rsrc_t out = uniform_buffer(recs, 8 * cap);
#pragma unroll
        for (int t = 0; t < kRecRing / 4; t += kWave)
            if (t + lane < pieces) __builtin_amdgcn_raw_buffer_store_b128(from[t + lane], out, 8 * gone + 16 * (t + lane), 0, kPayloadStorePolicy);
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ void take(int i, const float4& f, uint32_t wa, uint32_t wb, bool even)
    {
        const float up = pend;
        pend = mult[i + 1 < n ? i + 1 : i];
        const float a = EpiMaxAbs::max_abs4(f);
        if (even) {
            top = a;
        } else {
            const uint32_t m = pair_max_nonneg_bits(top, a, lane & 1);
            if (lane < 2) acc[i - 1 + lane] = m;
        }
        keep_signs(i, f);
        const bool c0 = fabsf(f.x) * up >= (float)(wa & 0xFFFFu), c1 = fabsf(f.y) * up >= (float)(wa >> 16);
        const bool c2 = fabsf(f.z) * up >= (float)(wb & 0xFFFFu), c3 = fabsf(f.w) * up >= (float)(wb >> 16);
        const uint64_t m0 = __builtin_amdgcn_ballot_w64(c0), m1 = __builtin_amdgcn_ballot_w64(c1);
        const uint64_t m2 = __builtin_amdgcn_ballot_w64(c2), m3 = __builtin_amdgcn_ballot_w64(c3);
        if ((m0 | m1 | m2 | m3) != 0 && count <= cap) {
            const uint32_t place = ((uint32_t)i << 8) | (4u * (uint32_t)lane);
            append(m0, c0, f.x, wa & 0xFFFFu, place);
            append(m1, c1, f.y, wa >> 16, place + 1u);
            append(m2, c2, f.z, wb & 0xFFFFu, place + 2u);
            append(m3, c3, f.w, wb >> 16, place + 3u);
            if (count - gone >= kRecRing / 2) {
                send(kRecRing / 4);
                gone += kRecRing / 2;
            }
        }
    }
    __device__ __forceinline__ void finish()
    {
        if (n & 1) {
            const uint32_t m = wave_max_nonneg_bits(top);
            if (lane == 0) acc[n - 1] = m;
        }
        if (count <= cap) send((count - gone + 1) / 2);
    }
};

// a block's largest magnitudes go to the bounds that lie below them
__device__ __forceinline__ void raise_bounds(const SketchArgs& a, const uint32_t* acc, int lane)
{
    asm volatile("" ::: "memory");  // the lanes read what others have written
    for (int i = lane; i < a.n; i += kWave) {
        const uint32_t m = __hip_atomic_load(a.run_max + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (acc[i] > m) (void)__hip_atomic_fetch_max(a.run_max + i, acc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("" ::: "memory");
}

// Largest-magnitude scales.  The largest magnitudes of the sample, and then of the blocks that are done, bound the scales from
// below, closer and closer as the pass goes on.  They are kept in the first row of the scale pass's array, which is also
// what the scales are taken from in the end; a block reads the row, and hands in only what lies above it.  What the values are
// like decides whether that pays, and the sample tells before (k_sketch_bounds_max): where it does not, this kernel returns at
// once and the scale pass runs instead.
// What bounds it: stores among reads, as in k_sketch.  64 workers x 25.6 M, three bits on average, heavy tails (t, three
// degrees), cyclic: 1330-1360 us, of which the bare row walk would be 960; some 450 records in a block (343 with the final
// scales as bounds, 2050 with the sample's); interval code 1400-1430.  Whole step 2338 us with two reads (scale pass 940, quantize pass
// 1390), 1755-1785 with one: sample 10, bounds 6, the scale pass that returns 5, this kernel, finalize 6, k_resolve 364-374, the quantize
// pass that finds nothing left 7.  One kernel with both passes: 2384 us for 2374 where values are alike (its registers and LDS are the
// sketch's), and with the first blocks of all in place of a sample 2123.
template <int S>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(S == 0 || S == kStreamDriver ? 1 : 4, S == 0 || S == kStreamDriver ? 8 : 4))) void k_sketch_max(
    const float* __restrict__ G, const int* __restrict__ row_ptr, const int* __restrict__ col,
    const float* __restrict__ val, const uint32_t* __restrict__ full, SketchArgs a, BitList in)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds_sketch_max[];
    if (load_uniform(full) > a.sk.limit) return;  // G is read twice
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t block = (int64_t)blockIdx.x * kSegBlocks + wave;
    const int64_t base = block * (int64_t)kBlockCoords;
    if (base >= a.d) {
        if (lane == 0) a.sk.counts[block] = 0;
        return;
    }
    uint32_t* slice = lds_sketch_max + wave * (sketch_max_lds_bytes(a.n) / 16);
    uint2* ring = reinterpret_cast<uint2*>(slice);
    uint32_t* plane = slice + 2 * kRecRing;
    uint32_t* acc = plane + 4 * a.sk.chunks * kWave;
    float* mult = reinterpret_cast<float*>(acc + a.n);
    for (int i = lane; i < a.n; i += kWave) {
        const uint32_t m = __hip_atomic_load(a.run_max + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float q = inv16_of(__uint_as_float(m), in.bits[i]);
        mult[i] = q > 0.f ? q : __builtin_inff();  // no bound, or a quotient beyond binary32
    }
    asm volatile("" ::: "memory");  // the lanes read what others have written
    const LaneCoords lc = lane_coords(base, lane, a.d);
    EpiSketchMax epi{{a.key0, a.key1, a.step_lo, a.step_hi, plane, a.n, lane, (uint32_t)((base + 4 * lane) >> 2)},
                     mult, acc, ring, a.sk.recs + block * (int64_t)a.sk.cap, a.sk.cap, 0, 0, 0.f, mult[0]};
    encode_block<S>(G + base, a.ldg, a.n, a.k, CsrView{row_ptr, col, val, a.win, a.stream, (int64_t)a.k * a.d <= kKeepElements}, lc, epi);
    epi.finish();
    store_plane(a, block, plane, lane);
    if (lane == 0) a.sk.counts[block] = epi.count <= a.sk.cap ? epi.count : -1;
    raise_bounds(a, acc, lane);
}

template <int S>
static hipError_t launch_sketch_max_s(const float* G, const CodeDev& code, const SketchArgs& a, const BitList& bits, hipStream_t stream)
{
    hipLaunchKernelGGL((k_sketch_max<S>), dim3((unsigned)((a.d + 1023) / 1024)), dim3(kWgThreads), sketch_max_lds_bytes(a.n), stream,
                       G, code.row_ptr, code.col, code.val, a.sk.state + 2, a, bits);
    return hipGetLastError();
}

template <int S>
static hipError_t launch_sketch_s(const float* G, const CodeDev& code, const SketchArgs& a, hipStream_t stream)
{
    hipLaunchKernelGGL((k_sketch<S>), dim3((unsigned)((a.d + 1023) / 1024)), dim3(kWgThreads), sketch_lds_bytes(a.n, a.sk.cap),
                       stream, G, code.row_ptr, code.col, code.val, a.sk.lo_mult, a);
    return hipGetLastError();
}

}  // namespace agc
