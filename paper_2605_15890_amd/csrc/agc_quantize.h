// K2 of the worker side: streaming encode + stochastic quantize + bit-pack (+ the fused estimate).
// Template code only; agc_quantize_b<0|1|2><s|m>.hip instantiate it for the three ways a block gets
// its multiplier and for one or several fills of the staging area, so that the sets of kernels
// compile in parallel.
#pragma once

#include "agc_device.h"
#include "agc_kernels.h"

namespace agc {

// =======================================================================================
// K2  encode + stochastic quantize + bit-pack
// =======================================================================================
struct QuantArgs {
    int64_t ldg;
    int n, k;
    int64_t d;
    uint32_t key0, key1, step_lo, step_hi;
    float* scales;  // bucket-wise scales only: n x nb
    int64_t nb;
    float* ghat;    // fused step only
    const WindowRec* win;  // monotone-interval codes only; filled in by the launcher
    const StreamRec* stream;  // codes that stream_records takes; likewise
    int stage_bits;        // bit-widths of the fullest fill of the staging area: at most stage_limit(), kPartBits with parts
    int stage_fills;       // how many fills the workers need: 1 unless the widths sum to more than that; always 1 with parts
    const uint8_t* block_layer;  // layer-wise scales only: the layer of every block; wq is then [layer][n]
    unsigned wg_first;     // the workgroups take the groups of four blocks from here upwards and then from 0; 0 with parts
    bool parts;            // short vectors: one block per workgroup, its workers shared among the waves
    // not null: only the groups of four blocks that k_resolve has left (agc_sketch.h): all of them if left_state[0] is not 0,
    // else the first left_state[1] of the list; never with parts
    const uint32_t* left_state;
    const uint32_t* left;
};

typedef __attribute__((address_space(1))) uint32_t global_u32;  // a pointer known to be device memory
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // one 16-byte piece of a stream

// Waves (= 256-coordinate blocks) per workgroup of the quantize pass.  A worker's codes leave in
// pieces of 32 * kQuantWaves * b contiguous bytes; the staging area grows by the same factor.
#ifndef AGC_K2_WG_WAVES
#define AGC_K2_WG_WAVES 4
#endif
constexpr int kQuantWaves = AGC_K2_WG_WAVES;
constexpr int kQuantThreads = kWave * kQuantWaves;

static_assert(kQuantWaves % 4 == 0 && kQuantWaves <= 16, "the per-worker table counts pieces for four waves");
static_assert(kParts == kQuantWaves, "a workgroup has four waves in either form");

// LDS staging area of a workgroup, in 16-byte pieces: 2 * blocks * bits pieces per worker
// (the blocks of the workgroup, 2 * bits pieces each), plus one piece that takes the zero bits the
// packer spills past a block's last word
__host__ __device__ constexpr int stage_pieces(int stage_bits, int blocks) { return 2 * blocks * stage_bits + 1; }

// raw buffer descriptor, last word: 32-bit untyped data format of this target; the bounds check is
// on the byte offset against num_records (stride 0)
constexpr int kBufferRsrcFlags = 0x00020000;
// cache-policy operand of the payload stores: bit 1 = non-temporal, bit 4 = sc1 (written through to
// memory), bit 0 = sc0.  Measured on the metric workload: plain 1.50 ms, sc0 1.51, sc1 1.45,
// non-temporal 1.42, non-temporal + sc1 1.41.
#ifndef AGC_PAYLOAD_POLICY
#define AGC_PAYLOAD_POLICY 18
#endif
constexpr int kPayloadStorePolicy = AGC_PAYLOAD_POLICY;

// cache-policy operand of the store of the fused estimate: sc1 alone (written through).  Next to
// the payload stores: plain 1.41-1.42 ms, non-temporal 1.43, sc1 1.40-1.41.
#ifndef AGC_ESTIMATE_POLICY
#define AGC_ESTIMATE_POLICY 16
#endif
constexpr int kEstimateStorePolicy = AGC_ESTIMATE_POLICY;

// buffer descriptor over `bytes` bytes at a wave-uniform address (the hardware drops accesses at
// offsets >= bytes).  The two halves of the address go through readfirstlane as unsigned words:
// the builtin returns a signed int, and a sign-extended low word would corrupt the high one.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_buffer(const void* p, int bytes)
{
    const uint64_t bits = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)bits);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(bits >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((char*)(((uint64_t)hi << 32) | (uint64_t)lo), 0,
                                             __builtin_amdgcn_readfirstlane(bytes), kBufferRsrcFlags);
}

// One rounding decision (Sec. II-B): T is the grid position scaled by 2^16; the cell is
// T >> 16, the low 16 bits are the first 16 bits of the round-up probability, compared with
// the 16-bit primary draw; equality is a tie, resolved later by a secondary draw.
__device__ __forceinline__ uint32_t round_primary(float T, uint32_t u16, uint32_t L, bool& tie)
{
    const uint32_t Ti = (uint32_t)T;
    tie = (u16 == (Ti & 0xFFFFu));
    // up <=> u16 < Fi <=> Fi + (0xFFFF - u16) carries into bit 16: one add and one shift
    const uint32_t level = (Ti + (0xFFFFu - u16)) >> 16;
    return level < L ? level : L;
}

// the same decision for a coordinate whose primary draw tied: U < (Fi+g)/2^16 <=> r2 < g*2^32
__device__ __forceinline__ uint32_t round_tied(float T, uint32_t r2, uint32_t L)
{
    const uint32_t Ti = (uint32_t)T;
    const float g = T - (float)Ti;
    const uint32_t up = ((double)r2 < (double)g * 4294967296.0) ? 1u : 0u;
    const uint32_t level = (Ti >> 16) + up;
    return level < L ? level : L;
}

template <bool ONEBIT>
__device__ __forceinline__ float grid_pos(float f, float inv)
{
    if (ONEBIT) return fmaxf(fmaf(f, inv, 32768.0f), 0.0f);
    return fabsf(f) * inv;
}

// The waves of a workgroup write out a fill of its staging area, workers first..last, which they share.  A worker's 2 * kBlocks
// * b pieces leave as one store of contiguous bytes through a buffer descriptor that covers exactly the bytes of the
// stream that exist, so the hardware's range check drops the pieces past the end of the vector.  Pieces are handed back
// zeroed.  wg_groups: 128-code groups of the workgroup's blocks that exist.
template <int kBlocks>
__device__ __forceinline__ void store_fill(uint32_t* stage, const WorkerQ* wq, int first, int last, int wave, int lane,
                                           int64_t wg, int wg_groups)
{
    u32x4_t* pieces = reinterpret_cast<u32x4_t*>(stage);
    for (int j = first + wave; j <= last; j += kQuantWaves) {
        const WorkerQ w = load_uniform(wq + j);
        const int b = (int)w.bits;
        const int np = 2 * kBlocks * b;  // pieces of this worker in the area
        const __amdgpu_buffer_rsrc_t rsrc = uniform_buffer(
            (const char*)w.codes + (uint64_t)wg * (uint64_t)(32 * kBlocks * b), 16 * b * wg_groups);
        const uint32_t at = w.stage_piece * (uint32_t)kBlocks / 4u;  // the table counts for four blocks
        for (int off = 0; off < np; off += kWave) {
            const int piece = off + lane;
            u32x4_t v = u32x4_t{0u, 0u, 0u, 0u};
            if (piece < np) {
                u32x4_t* sp = pieces + (at + (uint32_t)piece);
                v = *sp;
                *sp = u32x4_t{0u, 0u, 0u, 0u};
            }
            // lanes with piece >= np lie at or past the worker's bytes >= valid_bytes: dropped by the range check
#ifndef AGC_ABLATE_STORES
            __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, 16 * piece, 0, kPayloadStorePolicy);
#endif
        }
    }
}

// BUCKET 0: the worker's multiplier comes from the table (one scale per vector).
// BUCKET 1 / 2: one scale per 256-coordinate block, derived here from the block itself (largest
// magnitude / Euclidean norm), stored by lane 0, and turned into the multiplier with one binary32
// division (Sec. II-B names the bucket-wise extension; this is its single-pass form).
// FUSE: the pass also accumulates the master's estimate (Sec. II-A aggregation) from the codes it
// has just formed: arrived workers in ascending order, one fused multiply-add each from 0, the
// arithmetic of the stand-alone decode kernel, so both give the same bits.
// Payload path: a worker's codes are not stored when they are formed.  Every wave ORs its block's
// 8b words into the workgroup's LDS staging area (worker-major, then block, so that the four
// blocks of a worker lie in stream order); when the area is full, or after the last worker, the
// workgroup meets at a barrier and writes each worker's 128*b bytes as one contiguous, line-aligned
// piece of its stream.  Stores of 64..96 bytes per wave and worker, as a wave alone would issue
// them, reach memory as partial lines and cost several times their bytes on this memory system.
// MULTI: the workers need more than one fill of the area, so it is also written out between
// workers, inside the streaming loop.  Without MULTI (the common case: widths sum to at most
// stage_limit(), 319 without bucket-wise scales, or kPartBits with PARTS) the loop over the workers
// contains no store at all and the kernel writes the area out once, after the loop; the encode
// drivers then keep their rolling prefetch.
// PARTS: short vectors.  The workgroup has one block, its waves share the workers (encode_block_part); the
// estimate needs them in ascending order and is formed from the staged codes by the kernel (staged_estimate).
template <int BUCKET, bool FUSE, bool MULTI, bool PARTS>
struct EpiQuant {
    static constexpr int kBlocks = PARTS ? 1 : kQuantWaves;  // of the workgroup
    static constexpr bool kStoresPerWorker = MULTI;  // stores inside the worker loop (a flush between workers)
    static constexpr bool kWantsZeros = BUCKET != 0;  // else codes4 drops the codes of coordinates >= d, and nothing else counts them
    static constexpr int kPrefetchRows = AGC_PREFETCH_ROWS;
    const WorkerQ* __restrict__ wq;
    uint32_t key0, key1, step_lo, step_hi;
    uint32_t* stage;     // the workgroup's LDS staging area, all zero between fills
    float* stage_scales; // bucket-wise scales: [n][kBlocks] floats behind the staging area
    int lane;
    int wave;
    int blk;             // this wave's block inside the workgroup
    int n;               // workers
    int64_t wg;          // index of the workgroup = index of its group of four blocks
    int wg_groups;       // 128-code groups of the workgroup's blocks that exist in the streams (1..2*kBlocks)
    int64_t block;       // index of this wave's 256-coordinate block
    uint32_t ctr0;       // m >> 2 of this lane's coordinates
    int nvalid;
    bool wave_ragged;    // wave-uniform: some lane has coordinates >= d
    uint32_t keep[4];       // the Philox block of a pair: two words of the even worker, two of the odd one
    float* scales;          // bucket-wise scales: n x nb
    int64_t nb;
    int group_first;        // first worker of the fill that is being staged
    float acc[4];           // fused step: this lane's four coordinates of the estimate
    WorkerQ pend;           // record of the worker that comes next, requested one worker early
    // bucket-wise scales: the even worker of a pair, or held_i < 0
    float4 held;
    WorkerQ held_q;
    int held_i;

    // The workgroup writes out the fill that ends with worker `last`.  Every wave of the
    // workgroup calls this for the same workers in the same order (also a wave whose block lies
    // past the end of the vector), so the barriers match.
    __device__ __forceinline__ void flush_fill(int last)
    {
        __syncthreads();
        store_fill<kBlocks>(stage, wq, group_first, last, wave, lane, wg, wg_groups);
        group_first = last + 1;
        if (last + 1 < n) {
            __syncthreads();  // the area is reused by the next fill
        } else if (BUCKET != 0) {
            // after the last worker: the scales of all workers for the workgroup's blocks, one run of
            // kBlocks floats per worker (the barrier above made every wave's entries visible)
            const int64_t first_block = wg * kBlocks;
            const int have = nb - first_block >= kBlocks ? kBlocks : (int)(nb - first_block);
            for (int t = wave * kWave + lane; t < n; t += kQuantThreads) {
                __attribute__((address_space(1))) float* dst =
                    (__attribute__((address_space(1))) float*)scales + ((int64_t)t * nb + first_block);
                if (kBlocks > 1 && have == kBlocks) {  // one run per worker, dword-aligned (a row of scales starts anywhere)
                    typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
                    for (int u = 0; u + 3 < kBlocks; u += 4)
                        *(__attribute__((address_space(1))) f32x4_a4*)(dst + u) =
                            f32x4_a4{stage_scales[t * kBlocks + u], stage_scales[t * kBlocks + u + 1],
                                     stage_scales[t * kBlocks + u + 2], stage_scales[t * kBlocks + u + 3]};
                } else {
#pragma unroll
                    for (int u = 0; u < kBlocks; ++u)
                        if (u < have) dst[u] = stage_scales[t * kBlocks + u];
                }
            }
        }
    }

    // a wave without a block (past the end of the vector) still takes part in every flush
    __device__ __forceinline__ void flush_only()
    {
        for (int i = 0; i < n; ++i) {
            const WorkerQ w = load_uniform(wq + i);
            if (w.flush) flush_fill(i);
        }
    }

    // The scales of workers i and i + 1 in this block and the multipliers num / scale, both at once: the even lanes have
    // the first worker's, the odd lanes the second's, after one exchange, so that the rest of the reduction, the square
    // root and the division are paid once.  Whole steps, a worker at a time | in pairs, us: Euclidean 64 x 5.4 M 406 | 346,
    // 32 x 11.7 M 419 | 374, max-abs 345 | 319 and 349 | 333, 16 x 1 M 23.5 | 23.3 (64 x 25.6 M 1469 | 1458: stores among
    // reads bound that one).  num = L * 2^16 (2^15 for a one-bit worker) comes with the worker's record.
    __device__ __forceinline__ void block_multipliers(int i, const float4& f0, const float4& f1, float num0, float num1,
                                                      bool two, float (&scale)[2], float (&inv)[2])
    {
        const bool odd = lane & 1;
        float s;
        if (BUCKET == 1) {
            const float a = fmaxf(fmaxf(fabsf(f0.x), fabsf(f0.y)), fmaxf(fabsf(f0.z), fabsf(f0.w)));
            const float b = fmaxf(fmaxf(fabsf(f1.x), fabsf(f1.y)), fmaxf(fabsf(f1.z), fabsf(f1.w)));
            s = __uint_as_float(pair_max_nonneg_bits(a, b, odd));
        } else {
            // squares are exact in binary64: the fused sums round as the plain ones do
            const double x0 = f0.x, x1 = f0.y, x2 = f0.z, x3 = f0.w, y0 = f1.x, y1 = f1.y, y2 = f1.z, y3 = f1.w;
            const double a = fma(x0, x0, x1 * x1) + fma(x2, x2, x3 * x3), b = fma(y0, y0, y1 * y1) + fma(y2, y2, y3 * y3);
            double v = exchange_pair<kDppQuadSwap1>(a, b, odd);
            v = v + dpp_f64<kDppQuadSwap2>(v);
            s = (float)sqrt(exchange_halves(exchange_quads(v)));
        }
        // the block's scales wait in LDS next to the codes ([worker][block of the workgroup]) and
        // leave with the last flush: 4-byte stores scattered over n rows cost far more than their bytes
        if (lane < (two ? 2 : 1)) stage_scales[(i + lane) * kBlocks + blk] = s;
        float q = (odd ? num1 : num0) / s;       // correctly rounded binary32 division
        q = q <= 3.402823466e+38f ? q : 0.0f;    // scale == 0 gives +inf and ends here too
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            scale[t] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(s), t));
            inv[t] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(q), t));
        }
    }

    // the same for one worker
    __device__ __forceinline__ float block_multiplier(int i, const float4& f, float num, float& scale)
    {
        if (BUCKET == 1) {
            const float a = fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w)));
            scale = __uint_as_float(wave_max_nonneg_bits(a));
        } else {
            const double x0 = f.x, x1 = f.y, x2 = f.z, x3 = f.w;
            const double s01 = x0 * x0 + x1 * x1;
            const double s23 = x2 * x2 + x3 * x3;
            scale = (float)sqrt(wave_butterfly_add(s01 + s23));
        }
        if (lane == 0) stage_scales[i * kBlocks + blk] = scale;
        const float q = num / scale;
        return q <= 3.402823466e+38f ? q : 0.0f;
    }

    // four rounding decisions; only the grid position differs between the regular grid
    // (b >= 2) and the two-point grid of a one-bit worker
    __device__ __forceinline__ void codes4(int i, const float4& f, float inv, int b, uint32_t wa,
                                           uint32_t wb, uint32_t (&c)[4], uint32_t (&lev)[4])
    {
        const float fv[4] = {f.x, f.y, f.z, f.w};
        const uint32_t u[4] = {wa & 0xFFFFu, wa >> 16, wb & 0xFFFFu, wb >> 16};
        const uint32_t L = (b >= 2) ? ((1u << (b - 1)) - 1u) : 1u;
        const uint32_t signbit = (b >= 2) ? (1u << (b - 1)) : 0u;
        bool tie[4];
        float T[4];
#ifdef AGC_ABLATE_QUANT  // measurement build: no rounding arithmetic, codes are arbitrary bits
#pragma unroll
        for (int q = 0; q < 4; ++q) lev[q] = c[q] = (__float_as_uint(fv[q]) >> 9) & L;
        (void)tie; (void)T; (void)u; (void)signbit; (void)inv;
        return;
#endif
        if (b >= 2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) T[q] = grid_pos<false>(fv[q], inv);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) T[q] = grid_pos<true>(fv[q], inv);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] = round_primary(T[q], u[q], L, tie[q]);
        if (__any(tie[0] | tie[1] | tie[2] | tie[3])) {  // about one wave pass in 250
            uint32_t r2[4];
            philox4x32_10(ctr0, 0x80000000u | (uint32_t)i, step_lo, step_hi, key0, key1, r2);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (tie[q]) c[q] = round_tied(T[q], r2[q], L);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) lev[q] = c[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] |= (__float_as_uint(fv[q]) >> ((32 - b) & 31)) & signbit;
        if (wave_ragged) {  // codes of coordinates >= d are zero padding
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q >= nvalid) c[q] = 0u;
        }
    }

    // the worker's parity known at compile time (ring and gather drivers)
    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f)
    {
        if (EVEN) draw(i);
        if constexpr (BUCKET == 0) {
            finish(i, f, EVEN ? keep[0] : keep[2], EVEN ? keep[1] : keep[3]);
        } else {
            if (EVEN) hold(i, f);
            else pair(i - 1, held, f, true);
        }
    }

    // the worker's parity known only at run time (window driver); workers still come in
    // ascending order, so an odd worker finds the second half of its pair's Philox block.  One worker at a time with
    // bucket-wise scales too: pairs double the code at every ring position (W = 4, 32 workers x 262 144, Euclidean
    // 27.8 us, in pairs 29.1, in pairs with the two workers in a loop 30.5)
    __device__ __forceinline__ void worker_any(int i, const float4& f)
    {
        uint32_t wa = keep[2], wb = keep[3];
        if ((i & 1) == 0) {  // wave-uniform
            draw(i);
            wa = keep[0];
            wb = keep[1];
        }
        finish(i, f, wa, wb);
    }

    __device__ __forceinline__ void draw(int i)
    {
        philox4x32_10(ctr0, (uint32_t)i >> 1, step_lo, step_hi, key0, key1, keep);
    }

    // bucket-wise scales: the first worker of a pair waits for the second
    __device__ __forceinline__ void hold(int i, const float4& f)
    {
        held = f;
        held_q = pend;
        held_i = i;
        pend = load_uniform(wq + (i + 1 < n ? i + 1 : i));
    }
    __device__ __forceinline__ void pair(int i, const float4& f0, const float4& f1, bool two)
    {
        const WorkerQ q0 = held_q, q1 = pend;
        held_i = -1;
        pend = load_uniform(wq + (i + 2 < n ? i + 2 : n - 1));
        float scale[2], inv[2];
        block_multipliers(i, f0, f1, q0.inv16, q1.inv16, two, scale, inv);
        emit(i, f0, q0, inv[0], scale[0], keep[0], keep[1]);
        if (two) emit(i + 1, f1, q1, inv[1], scale[1], keep[2], keep[3]);
    }
    // after the last worker: one that is still waiting for another
    __device__ __forceinline__ void finish_pairs()
    {
        if constexpr (BUCKET != 0)
            if (held_i >= 0) pair(held_i, held, held, false);
    }

    __device__ __forceinline__ void finish(int i, const float4& f, uint32_t wa, uint32_t wb)
    {
        // wave-uniform scalar reads; workers come in ascending order, so the record of this one
        // was requested while the previous one was quantized
        const WorkerQ q = pend;
        pend = load_uniform(wq + (i + 1 < n ? i + 1 : i));
        float scale = 0.f;
        const float inv = BUCKET == 0 ? q.inv16 : block_multiplier(i, f, q.inv16, scale);
        emit(i, f, q, inv, scale, wa, wb);
    }

    __device__ __forceinline__ void emit(int i, const float4& f, const WorkerQ& q, float inv, float scale, uint32_t wa, uint32_t wb)
    {
        const int b = (int)q.bits;
        uint32_t c[4], lev[4];
        codes4(i, f, inv, b, wa, wb, c, lev);
        if constexpr (FUSE && !PARTS) {
            if (q.arrived) {  // wave-uniform
                const float coef = BUCKET == 0 ? q.coef : q.coef * scale;
                const float fv[4] = {f.x, f.y, f.z, f.w};
                // the decoded value: +-level (the level as a float with the sign bit of f), or +-1
                // for a one-bit worker; one fused multiply-add per coordinate either way
                float v[4];
                if (b >= 2) {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        v[t] = __uint_as_float(__float_as_uint((float)lev[t]) | (__float_as_uint(fv[t]) & 0x80000000u));
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = lev[t] ? 1.0f : -1.0f;
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[t] = fmaf(coef, v[t], acc[t]);
            }
        }

        // bit-pack: this lane's four codes start at bit lane*4b of the block's 256*b bits, the block's
        // 8b words start at piece q.stage_piece + wave*2b of the staging area
        const uint32_t bitpos = __umul24((uint32_t)lane, 4u * (uint32_t)b);
        uint32_t* slot = stage + 4u * (q.stage_piece * (uint32_t)kBlocks / 4u + (uint32_t)blk * 2u * (uint32_t)b) +
                         (bitpos >> 5);
        const uint32_t sh = bitpos & 31u;
#ifdef AGC_ABLATE_PACK
        if (c[0] + c[1] + c[2] + c[3] + sh == 0xFFFFFFF0u) atomicOr(slot, 1u);
        else
#endif
        if (b <= 8) {
            const uint32_t chunk = c[0] | (c[1] << b) | (c[2] << (2 * b)) | (c[3] << (3 * b));
            const uint64_t v = (uint64_t)chunk << sh;
            atomicOr(slot, (uint32_t)v);
            atomicOr(slot + 1, (uint32_t)(v >> 32));
        } else {
            const uint64_t chunk = (uint64_t)c[0] | ((uint64_t)c[1] << b) | ((uint64_t)c[2] << (2 * b)) |
                                   ((uint64_t)c[3] << (3 * b));
            const uint64_t v = chunk << sh;
            const uint32_t top = sh ? (uint32_t)(chunk >> (64 - sh)) : 0u;
            atomicOr(slot, (uint32_t)v);
            atomicOr(slot + 1, (uint32_t)(v >> 32));
            atomicOr(slot + 2, top);
        }
        if constexpr (MULTI) {
            if (q.flush) flush_fill(i);  // wave-uniform, and the same for every wave of the workgroup
        }
    }
};

// The fused estimate of short vectors: thread t forms coordinate t of the workgroup's block from the staged
// codes of all workers, arrived ones in ascending order, one fused multiply-add each - the arithmetic of the
// other forms.  Four workers' words are requested together.
template <int BUCKET>
__device__ __forceinline__ float staged_estimate(const WorkerQ* __restrict__ wq, const uint32_t* stage,
                                                 const float* stage_scales, int n)
{
    constexpr int kBatch = 4;
    const uint32_t t = threadIdx.x;
    float acc = 0.f;
    for (int e0 = 0; e0 < n; e0 += kBatch) {
        WorkerQ q[kBatch];
        uint32_t w0[kBatch], w1[kBatch];
        float sc[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) q[u] = load_uniform(wq + (e0 + u < n ? e0 + u : n - 1));
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t* p = stage + q[u].stage_piece + ((t * q[u].bits) >> 5);  // a quarter of the pieces, four words each
            w0[u] = p[0];
            w1[u] = p[1];
            sc[u] = BUCKET != 0 ? stage_scales[e0 + u < n ? e0 + u : n - 1] : 1.f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (e0 + u >= n || !q[u].arrived) continue;  // wave-uniform
            const uint32_t b = q[u].bits;
            const uint32_t code = __builtin_amdgcn_alignbit(w1[u], w0[u], (t * b) & 31u);
            const float coef = BUCKET == 0 ? q[u].coef : q[u].coef * sc[u];
            float v;
            if (b >= 2) {
                const uint32_t level = code & ((1u << (b - 1)) - 1u);
                v = __uint_as_float(__float_as_uint((float)level) | ((code << (32 - b)) & 0x80000000u));
            } else {
                v = (code & 1u) ? 1.0f : -1.0f;
            }
            acc = fmaf(coef, v, acc);
        }
    }
    return acc;
}

// LEFT: only the groups of blocks that k_resolve has left (an instance of its own: the test alone cost the others 0.3 us).
template <int S, int BUCKET, bool FUSE, bool MULTI, bool PARTS, bool LEFT = false>
// The compiler is told to plan for four waves per SIMD: with a register count just under the
// five-wave limit it otherwise schedules for five and gives up instruction-level parallelism;
// measured 1.45 ms against 1.51 ms on the metric workload (three: 1.51 ms).  The gather driver
// (S == 0) lives on occupancy instead and keeps the default.
#ifndef AGC_K2_WAVES
#define AGC_K2_WAVES 4
#endif
__global__ __launch_bounds__(kQuantThreads) __attribute__((amdgpu_waves_per_eu(S == 0 || S == kStreamDriver ? 1 : AGC_K2_WAVES, S == 0 || S == kStreamDriver ? 8 : AGC_K2_WAVES))) void k_quantize(const float* __restrict__ G,
                                                         const int* __restrict__ row_ptr,
                                                         const int* __restrict__ col,
                                                         const float* __restrict__ val,
                                                         const WorkerQ* __restrict__ wq, QuantArgs a)
{
    static_assert(!(MULTI && PARTS), "the parts of the workers meet in one fill");
    constexpr int kBlocks = PARTS ? 1 : kQuantWaves;
    // stage_pieces(a.stage_bits, kBlocks) pieces, then (bucket-wise scales) n * kBlocks floats
    extern __shared__ __attribute__((aligned(16))) uint32_t lds_stage[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform by construction
    const int lane = threadIdx.x % kWave;
    unsigned wg_index = blockIdx.x + a.wg_first;  // < 2 * grid <= 2^24
    if (wg_index >= gridDim.x) wg_index -= gridDim.x;
    if constexpr (LEFT) {
        // Workgroups go to the eight dies in turn.  The groups that are left may lie a multiple of eight apart (the first columns of
        // matrices), so the first workgroups take them from a list; while each looked after its own group, one die did all of
        // the work: 64 x 25.6 M, rows of 16384 whose first 256 values are 20 times the others, six bits, whole step
        // 3107 | 1950 us (two reads 2500).
        struct State { uint32_t all, count; };
        const State s = load_uniform(reinterpret_cast<const State*>(a.left_state));
        if (s.all == 0u) {
            if (blockIdx.x >= s.count) return;
            wg_index = load_uniform(a.left + blockIdx.x);
        }
    }
    const int64_t wg = wg_index;
    const int64_t block = PARTS ? wg : wg * kQuantWaves + wave;
    const int64_t base = block * (int64_t)kBlockCoords;
    {
        u32x4_t* pieces = reinterpret_cast<u32x4_t*>(lds_stage);
        const int np = stage_pieces(a.stage_bits, kBlocks);
        for (int p = threadIdx.x; p < np; p += kQuantThreads) pieces[p] = u32x4_t{0u, 0u, 0u, 0u};
    }
    __syncthreads();
    const int64_t groups_left = (a.d + 127) / 128 - 2 * kBlocks * wg;  // >= 1: the workgroup's first block exists
    const bool has_block = base < a.d;
    LaneCoords lc{};
    if (has_block) lc = lane_coords(base, lane, a.d);
    // layer-wise scales: the table of the block's layer (multiplier and decode weight differ from
    // layer to layer; bit-width, stream and staging place are the same in every table, so the
    // waves of a workgroup may hold different tables when they meet at a flush)
    if (a.block_layer && has_block) wq += (int64_t)__builtin_amdgcn_readfirstlane((int)a.block_layer[block]) * a.n;
    const int part = PARTS ? part_size(a.n) : 0;
    const int i0 = PARTS ? (wave * part < a.n ? wave * part : a.n) : 0, i1 = PARTS ? (i0 + part < a.n ? i0 + part : a.n) : a.n;
    float* stage_scales = reinterpret_cast<float*>(lds_stage + 4 * stage_pieces(a.stage_bits, kBlocks));
    EpiQuant<BUCKET, FUSE, MULTI, PARTS> epi{wq, a.key0, a.key1, a.step_lo, a.step_hi, lds_stage, stage_scales, lane, wave,
                               PARTS ? 0 : wave, a.n, wg,
                               groups_left >= 2 * kBlocks ? 2 * kBlocks : (int)groups_left, block, (uint32_t)((base + 4 * lane) >> 2),
                               lc.nvalid, lc.wave_ragged, {0u, 0u, 0u, 0u}, a.scales, a.nb, 0, {0.f, 0.f, 0.f, 0.f},
                               load_uniform(wq + (i0 < a.n ? i0 : 0)), make_float4(0.f, 0.f, 0.f, 0.f), WorkerQ{}, -1};
    if constexpr (PARTS) {  // every workgroup has its block
        encode_block_part<S>(G + base, a.ldg, a.k, CsrView{row_ptr, col, val, a.win}, lc, i0, i1, epi);
        epi.finish_pairs();
        if constexpr (FUSE) {
            __syncthreads();
            const float g = staged_estimate<BUCKET>(wq, lds_stage, stage_scales, a.n);
            if (base + (int64_t)threadIdx.x < a.d) a.ghat[base + threadIdx.x] = g;
        }
        epi.flush_fill(a.n - 1);  // its barrier: the codes have been read before the pieces are handed back
        return;
    }
    if (!has_block) {  // nothing to encode, but the other waves of the workgroup wait at the flushes
        if constexpr (MULTI) epi.flush_only();
        else epi.flush_fill(a.n - 1);
        return;
    }
    encode_block<S>(G + base, a.ldg, a.n, a.k, CsrView{row_ptr, col, val, a.win, a.stream, (int64_t)a.k * a.d <= kKeepElements}, lc, epi);
    epi.finish_pairs();
    if constexpr (!MULTI) epi.flush_fill(a.n - 1);  // the one fill: all workers, written out after the loop
    if constexpr (FUSE) {
        float* dst = a.ghat + base + 4 * lane;
        if (lc.nvalid == 4) {
            const __amdgpu_buffer_rsrc_t rs = uniform_buffer(a.ghat + base, 4 * kBlockCoords);
            __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{__float_as_uint(epi.acc[0]), __float_as_uint(epi.acc[1]),
                                                           __float_as_uint(epi.acc[2]), __float_as_uint(epi.acc[3])},
                                                   rs, 16 * lane, 0, kEstimateStorePolicy);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t < lc.nvalid) dst[t] = epi.acc[t];
        }
    }
}

template <int S, int BUCKET, bool MULTI>
static hipError_t launch_quantize_s(const float* G, const CodeDev& code, const Workspace& ws,
                                    const QuantArgs& args, hipStream_t stream)
{
    QuantArgs a = args;
    a.win = code.win;
    a.stream = code.stream;
    if (S < 0 && S != kStreamDriver && !a.win) return hipErrorInvalidValue;  // the window driver reads the records
    const int64_t nblocks = (a.d + kBlockCoords - 1) / kBlockCoords;
    const unsigned grid = (unsigned)((nblocks + kQuantWaves - 1) / kQuantWaves);
    if (a.stage_bits < 1 || a.stage_bits > (a.parts ? kPartBits : kStageBits)) return hipErrorInvalidValue;
    if (MULTI ? a.stage_fills < 2 : a.stage_fills != 1) return hipErrorInvalidValue;
    if constexpr (!MULTI && S != kStreamDriver) {
        if (a.parts) {
            const unsigned lds = 16u * (unsigned)stage_pieces(a.stage_bits, 1) + (BUCKET != 0 ? 4u * (unsigned)a.n : 0u);
            const dim3 g((unsigned)nblocks), b(kWave * kParts);
            if (a.ghat)
                hipLaunchKernelGGL((k_quantize<S, BUCKET, true, false, true>), g, b, lds, stream, G, code.row_ptr, code.col,
                                   code.val, ws.wq, a);
            else
                hipLaunchKernelGGL((k_quantize<S, BUCKET, false, false, true>), g, b, lds, stream, G, code.row_ptr,
                                   code.col, code.val, ws.wq, a);
            return hipGetLastError();
        }
    }
    a.wg_first = BUCKET == 0 ? first_group(a.d, grid) : 0u;
    const unsigned lds_bytes = 16u * (unsigned)stage_pieces(a.stage_bits, kQuantWaves) +
                               (BUCKET != 0 ? (unsigned)(sizeof(float) * kQuantWaves * a.n) : 0u);
    const dim3 g(grid), b(kQuantThreads);
    if constexpr (BUCKET == 0) {
        if (a.left) {
            if (a.ghat)
                hipLaunchKernelGGL((k_quantize<S, 0, true, MULTI, false, true>), g, b, lds_bytes, stream, G, code.row_ptr,
                                   code.col, code.val, ws.wq, a);
            else
                hipLaunchKernelGGL((k_quantize<S, 0, false, MULTI, false, true>), g, b, lds_bytes, stream, G, code.row_ptr,
                                   code.col, code.val, ws.wq, a);
            return hipGetLastError();
        }
    }
    if (a.ghat)
        hipLaunchKernelGGL((k_quantize<S, BUCKET, true, MULTI, false>), g, b, lds_bytes, stream, G, code.row_ptr, code.col,
                           code.val, ws.wq, a);
    else
        hipLaunchKernelGGL((k_quantize<S, BUCKET, false, MULTI, false>), g, b, lds_bytes, stream, G, code.row_ptr, code.col,
                           code.val, ws.wq, a);
    return hipGetLastError();
}

template <int BUCKET, bool MULTI>
static inline hipError_t launch_quantize_band(const float* G, const CodeDev& code, const Workspace& ws,
                                              const QuantArgs& a, hipStream_t stream)
{
    switch (code.band) {
        case 1: return launch_quantize_s<1, BUCKET, MULTI>(G, code, ws, a, stream);
        case 2: return launch_quantize_s<2, BUCKET, MULTI>(G, code, ws, a, stream);
        case 3: return launch_quantize_s<3, BUCKET, MULTI>(G, code, ws, a, stream);
        case 4: return launch_quantize_s<4, BUCKET, MULTI>(G, code, ws, a, stream);
        case 5: return launch_quantize_s<5, BUCKET, MULTI>(G, code, ws, a, stream);
        case 6: return launch_quantize_s<6, BUCKET, MULTI>(G, code, ws, a, stream);
        case 7: return launch_quantize_s<7, BUCKET, MULTI>(G, code, ws, a, stream);
        case 8: return launch_quantize_s<8, BUCKET, MULTI>(G, code, ws, a, stream);
        case -2: return launch_quantize_s<-2, BUCKET, MULTI>(G, code, ws, a, stream);
        case -4: return launch_quantize_s<-4, BUCKET, MULTI>(G, code, ws, a, stream);
        case -8: return launch_quantize_s<-8, BUCKET, MULTI>(G, code, ws, a, stream);
        default:
            return code.stream && !a.parts ? launch_quantize_s<kStreamDriver, BUCKET, MULTI>(G, code, ws, a, stream)
                                           : launch_quantize_s<0, BUCKET, MULTI>(G, code, ws, a, stream);
    }
}

// One entry point per instantiation unit (agc_quantize_b<BUCKET><s|m>.hip: the way a block gets its
// multiplier, and one fill or several), so that the sets of kernels compile in parallel.
#define AGC_QUANT_UNIT(NAME) \
    hipError_t NAME(const float* G, const CodeDev& code, const Workspace& ws, const QuantArgs& a, hipStream_t stream)
AGC_QUANT_UNIT(launch_quantize_band0s);
AGC_QUANT_UNIT(launch_quantize_band0m);
AGC_QUANT_UNIT(launch_quantize_band1s);
AGC_QUANT_UNIT(launch_quantize_band1m);
AGC_QUANT_UNIT(launch_quantize_band2s);
AGC_QUANT_UNIT(launch_quantize_band2m);

}  // namespace agc
