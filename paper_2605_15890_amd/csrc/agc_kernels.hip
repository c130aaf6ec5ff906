// gfx950 kernels of the approximate-gradient-coding hot path.
//
//   k_scale_pass      worker side, pass 1: stream G once, form f_i = sum_j a_ij g_j in registers
//                     (Sec. II-A) and reduce each worker's scale: running maxima in a small
//                     array (max-abs, also per layer), sums of squares per 1024-coordinate
//                     segment (Euclidean)
//   k_scale_finalize  the maxima, or a fixed-order reduction of the segment sums -> scale_i and
//   (.._layers)       the per-worker table (inv16_i, b_i, stream pointer) of the next pass
//   k_quantize        worker side, pass 2: stream G once more, re-form f_i, stochastic rounding
//                     on the grid {0,1/L,..,1} (Sec. II-B) with Philox draws, variable-width
//                     bit-packing, coalesced stores of the payload
//   k_decode_table    master side prologue: table of the arrived workers with their weights
//   k_decode          master side: masked dequantize + weighted sum (Sec. II-A aggregation)
//
// All of them are bandwidth/ALU streaming kernels; there is no dense contraction on this
// path, hence no MFMA.  Per-worker parameters are read with scalar loads from small device
// tables, never with vector loads, so that waiting for them does not drain the queue of
// outstanding row loads.
#include <mutex>

#include "agc_device.h"
#include "agc_kernels.h"
#include "agc_quantize.h"

namespace agc {

// =======================================================================================
// K1  scale pass
// =======================================================================================
// Pointers that the kernels only read are separate __restrict__ kernel parameters: that is
// what lets the compiler keep wave-uniform reads (code coefficients, per-worker tables) on the
// scalar unit even though the same kernel stores through other pointers.
struct ScaleArgs {
    int64_t ldg;
    int n, k;
    int64_t d;
    int64_t nseg;
    uint32_t* part_max;
    double* part_sq;
    const WindowRec* win;  // monotone-interval codes only
    const StreamRec* stream;     // codes that stream_records takes
    const uint8_t* block_layer;  // layer-wise scales only (max-abs): the layer of every block
    const int* seg_first;        // layer-wise Euclidean scales only: the segments of the layers
    const uint8_t* seg_blocks;
    const uint32_t* full;        // COND: nothing to do where this word is at most `limit` (the sketch serves the step)
    uint32_t limit;
};

// the same 32-bit word seen as device memory (store without address-space checks)
typedef __attribute__((address_space(1))) uint32_t global_word;

// epilogue for the Euclidean scale: levels 0 and 1 of the binary64 summation tree (lane value
// (x0^2+x1^2)+(x2^2+x3^2); exchange-add across the 64 lanes)
struct EpiSumSq {
    typedef double Part, Sum;
    static constexpr bool kStoresPerWorker = false;
    static constexpr bool kWantsZeros = true;
    static constexpr int kPrefetchRows = AGC_SCALE_PREFETCH_ROWS;
    double* acc;  // this wave's LDS slice [n]
    int lane;
    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f)
    {
        const double x0 = f.x, x1 = f.y, x2 = f.z, x3 = f.w;
        const double s01 = x0 * x0 + x1 * x1;
        const double s23 = x2 * x2 + x3 * x3;
        const double q = wave_butterfly_add(s01 + s23);
        if (lane == 0) acc[i] = q;
    }
    __device__ __forceinline__ void worker_any(int i, const float4& f) { worker<true>(i, f); }
};

// The norm's workgroups are the four blocks of a segment of its summation tree; the max-abs pass
// is free in its workgroup size (4 and 8 waves measured within 1 % of each other, 16 waves 2 %
// slower) and, with two blocks per wave, in its prefetch distance (2 to 8 rows within 1 %).
#ifndef AGC_SCALE_WAVES
#define AGC_SCALE_WAVES 8
#endif
#ifndef AGC_SCALE_PREFETCH_ROWS2
#define AGC_SCALE_PREFETCH_ROWS2 2  // rows ahead in the two-block ring: four loads in flight per lane
#endif
// below this many blocks the two-block form would leave compute units without a wave
// (256 units x 4 SIMDs x 5 resident waves of two blocks each, twice over)
constexpr int64_t kTwoBlockMin = 2 * 2 * 256 * 4 * 5;
// Euclidean scale: one workgroup per 1024-coordinate segment, one wave per 256-coordinate block of
// it.  The four block values of every worker meet in LDS and are combined in block order (level 2
// of the tree), which keeps the result independent of how the waves were scheduled.
// Max-abs scale: the maximum is exact and order-free.  A wave takes V neighbouring blocks (V = 2:
// both at once through the two-block register ring when they lie wholly inside the vector and the
// code has a ring driver, else one after the other) and folds its n maxima into the workgroup's
// LDS array with LDS atomics; the last wave of the workgroup to finish folds that array into one
// of kMaxSlots rows of a small array in memory ([slot][worker]) with one integer atomic-max
// instruction (bit patterns of non-negative floats order like the floats).  No wave waits for
// another, and the pass writes no partial results to memory (stores mixed into the read stream
// cost far more than their bytes on this memory system; even the atomics, performed in memory,
// cost 22 us at one per wave and worker).  The finalize kernel reads the rows and hands them back
// zeroed.
template <int S, int MODE, int WAVES, int V, bool COND = false>
__global__ __launch_bounds__(kWave * WAVES) void k_scale_pass(const float* __restrict__ G,
                                                              const int* __restrict__ row_ptr,
                                                              const int* __restrict__ col,
                                                              const float* __restrict__ val,
                                                              ScaleArgs a)
{
    static_assert(MODE == 1 || (WAVES == kSegBlocks && V == 1), "the norm's tree fixes four blocks per workgroup");
    static_assert(V == 1 || V == 2 || V == 4, "one, two or four blocks per wave");
    __shared__ double lds_acc[WAVES][kMaxWorkers];
    if constexpr (COND) {
        if (load_uniform(a.full) <= a.limit) return;
    }
    // the wave index is the same for all lanes: tell the compiler, so that everything derived
    // from it (block base, pointers) lives in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t seg = blockIdx.x;
    const int64_t blk = seg * WAVES + wave;  // max-abs: index of the wave's run of V blocks
    const int64_t base = blk * (int64_t)(V * kBlockCoords);
    const CsrView B{row_ptr, col, val, a.win, a.stream, (int64_t)a.k * a.d <= kKeepElements};

    double* accd = lds_acc[wave];
    uint32_t* accu = reinterpret_cast<uint32_t*>(lds_acc[wave]);
    if (MODE == 1) {
        // the workgroup's running maxima and the count of waves that have delivered theirs
        __shared__ uint32_t wg_max[kMaxWorkers];
        __shared__ uint32_t wg_done;
        for (int i = threadIdx.x; i < a.n; i += kWave * WAVES) wg_max[i] = 0u;
        if (threadIdx.x == 0) wg_done = 0u;
        __syncthreads();  // the only barrier: at the start, where no wave has anything to wait for
        EpiMaxAbs epi{accu, lane};
        // Layer-wise scales (Sec. II-B names the layer-wise granularity): layer l owns rows
        // l*kLayerSub .. l*kLayerSub+kLayerSub-1 of the slot array (several rows, so that the
        // workgroups that walk one layer at the same time do not all hit the same words).  The
        // workgroup's LDS array collects the layer of the workgroup's first block; a wave whose
        // blocks lie in another layer (a workgroup that straddles a boundary) hands its maxima to
        // that layer's row itself.
        const int64_t last_block = (a.d - 1) / kBlockCoords;
        const int64_t wg_first = (int64_t)blockIdx.x * (WAVES * V);
        const int layer0 = a.block_layer
                               ? __builtin_amdgcn_readfirstlane((int)a.block_layer[wg_first < last_block ? wg_first : last_block])
                               : 0;
        const int sub = (int)(blockIdx.x % kLayerSub);
        auto fold = [&](int layer) {  // accu[i] was written by this wave's lane 0
            if (layer == layer0) {
                for (int i = lane; i < a.n; i += kWave)
                    (void)__hip_atomic_fetch_max(wg_max + i, accu[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                uint32_t* dst = a.part_max + ((int64_t)layer * kLayerSub + sub) * a.n;
                for (int i = lane; i < a.n; i += kWave)
                    (void)__hip_atomic_fetch_max(dst + i, accu[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        };
        auto layer_of = [&](int64_t first_coord) {
            return a.block_layer ? __builtin_amdgcn_readfirstlane((int)a.block_layer[first_coord / kBlockCoords]) : 0;
        };
        if (base < a.d) {
            bool together = V > 1 && S != 0 && base + V * kBlockCoords <= a.d;
            if (together && a.block_layer) {  // all V blocks in one layer
                for (int u = 1; u < V; ++u)
                    together = together && layer_of(base + (int64_t)u * kBlockCoords) == layer_of(base);
            }
            if (together) {
                const LaneCoords lc = lane_coords(base, lane, a.d);  // every lane whole, in all V blocks
                if constexpr (S == kStreamDriver) encode_stream<RowN<V>>(G + base, a.ldg, a.k, B, lc, epi);
                else if constexpr (S > 0) encode_ring<S, AGC_SCALE_PREFETCH_ROWS2, RowN<V>>(G + base, a.ldg, a.k, val, lc, epi);
                else if constexpr (S < 0) encode_window<-S, AGC_SCALE_PREFETCH_ROWS2, RowN<V>>(G + base, a.ldg, a.k, B, lc, epi);
                fold(layer_of(base));
            } else {
                for (int u = 0; u < V; ++u) {
                    const int64_t b = base + (int64_t)u * kBlockCoords;
                    if (b < a.d) {
                        const LaneCoords lc = lane_coords(b, lane, a.d);
                        encode_block<S>(G + b, a.ldg, a.n, a.k, B, lc, epi);
                        fold(layer_of(b));
                    }
                }
            }
        }
        // Nobody waits for anybody: a wave that is done makes sure its maxima have reached wg_max
        // (release fence: the wave's LDS operations have completed) and adds itself to the count;
        // the wave that finds itself last hands the workgroup's maxima to the slot array - one
        // memory-side atomic per worker and workgroup instead of one per wave.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        uint32_t before = 0u;
        if (lane == 0) before = __hip_atomic_fetch_add(&wg_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        before = (uint32_t)__builtin_amdgcn_readfirstlane((int)before);
        if (before == (uint32_t)(WAVES - 1)) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            uint32_t* dst = a.part_max + (a.block_layer ? (int64_t)layer0 * kLayerSub + sub
                                                        : ((int64_t)blockIdx.x & (kMaxSlots - 1))) * a.n;
            for (int i = lane; i < a.n; i += kWave) {
                const uint32_t m = __hip_atomic_load(wg_max + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (m != 0u) (void)__hip_atomic_fetch_max(dst + i, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        return;
    }
    // Euclidean scale per layer: segment `seg` is the table's run of up to four blocks (the tree of
    // a layer starts at the layer's first block); a wave past the run contributes nothing
    int64_t sq_base = base;
    bool sq_has = base < a.d;
    if (a.seg_first) {
        sq_base = ((int64_t)a.seg_first[seg] + wave) * (int64_t)kBlockCoords;
        sq_has = wave < (int)a.seg_blocks[seg];
    }
    if (sq_has) {
        const LaneCoords lc = lane_coords(sq_base, lane, a.d);
        EpiSumSq epi{accd, lane};
        encode_block<S>(G + sq_base, a.ldg, a.n, a.k, B, lc, epi);
    } else {  // a block past the end of the vector (or of the layer's last segment) contributes nothing
        for (int i = lane; i < a.n; i += kWave) accd[i] = 0.0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < a.n; i += kWave * WAVES) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum = sum + lds_acc[w][i];
        // [segment][worker]: one coalesced row per workgroup, non-temporal (a plain store costs the
        // pass 30 us more: the dirty lines leave the cache in the middle of the read stream)
        __builtin_nontemporal_store(sum, a.part_sq + seg * (int64_t)a.n + i);
    }
}

// Short vectors: the waves of a workgroup share the workers of a block, kParts ways.  A wave alone on its
// SIMD issues one instruction in about five cycles, and walking over 64 workers one after the other takes it
// longer than the memory needs for everything; the rows at the seams of the parts are read twice, which is
// nothing at these sizes.  Max-abs: one block per workgroup, and every wave hands its maxima to the slot
// array itself.  Euclidean: the four blocks of a segment, sixteen waves.
template <int S, int MODE>
__global__ __launch_bounds__(kWave * (MODE == 1 ? kParts : kParts * kSegBlocks)) void k_scale_pass_parts(
    const float* __restrict__ G, const int* __restrict__ row_ptr, const int* __restrict__ col,
    const float* __restrict__ val, ScaleArgs a)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const CsrView B{row_ptr, col, val, a.win};
    const int size = part_size(a.n);
    const int i0 = (MODE == 1 ? wave : wave / kSegBlocks) * size;
    const int i1 = i0 + size < a.n ? i0 + size : a.n;
    if constexpr (MODE == 1) {
        __shared__ uint32_t lds_max[kMaxWorkers];
        const int64_t blk = blockIdx.x;
        const int64_t base = blk * kBlockCoords;
        const LaneCoords lc = lane_coords(base, lane, a.d);
        EpiMaxAbs epi{lds_max, lane};
        encode_block_part<S>(G + base, a.ldg, a.k, B, lc, i0, i1, epi);
        const int64_t slot = a.block_layer ? (int64_t)a.block_layer[blk] * kLayerSub + blk % kLayerSub : blk & (kMaxSlots - 1);
        for (int i = i0 + lane; i < i1; i += kWave) {  // written by this wave's lane 0
            const uint32_t m = lds_max[i];
            if (m != 0u)
                (void)__hip_atomic_fetch_max(a.part_max + slot * a.n + i, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else {
        __shared__ double lds_sq[kSegBlocks][kMaxWorkers];
        const int64_t seg = blockIdx.x;
        const int b = wave % kSegBlocks;
        int64_t base = (seg * kSegBlocks + b) * (int64_t)kBlockCoords;
        bool has = base < a.d;
        if (a.seg_first) {
            base = ((int64_t)a.seg_first[seg] + b) * (int64_t)kBlockCoords;
            has = b < (int)a.seg_blocks[seg];
        }
        if (has) {
            const LaneCoords lc = lane_coords(base, lane, a.d);
            EpiSumSq epi{lds_sq[b], lane};
            encode_block_part<S>(G + base, a.ldg, a.k, B, lc, i0, i1, epi);
        } else {
            for (int i = i0 + lane; i < i1; i += kWave) lds_sq[b][i] = 0.0;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < a.n; i += kWave * kParts * kSegBlocks) {
            double sum = 0.0;
#pragma unroll
            for (int w = 0; w < kSegBlocks; ++w) sum = sum + lds_sq[w][i];
            __builtin_nontemporal_store(sum, a.part_sq + seg * (int64_t)a.n + i);
        }
    }
}

// What the finalize kernel hands back zeroed: rows of the max-abs slot array, and the sketch's cost of the sampled blocks (state
// null: there is none).  Creation does it with a memset; this kernel serves a call that follows one whose launches failed half-way.
__global__ __launch_bounds__(kWgThreads) void k_scale_clear_slots(uint32_t* slots, int count, uint32_t* state)
{
    const int t = blockIdx.x * kWgThreads + threadIdx.x;
    if (t < count) slots[t] = 0u;
    if (t == 0 && state) state[2] = 0u;
}

hipError_t launch_scale_clear_slots(int n, const Workspace& ws, uint32_t* state, hipStream_t stream)
{
    const int count = n * ws.max_rows;
    hipLaunchKernelGGL(k_scale_clear_slots, dim3((count + kWgThreads - 1) / kWgThreads), dim3(kWgThreads), 0, stream,
                       ws.part_max, count, state);
    return hipGetLastError();
}

#ifndef AGC_SCALE_BLOCKS_PER_WAVE
#define AGC_SCALE_BLOCKS_PER_WAVE 2
#endif
template <int S, int V>
static void launch_scale_max(const float* G, const CodeDev& code, const ScaleArgs& a, hipStream_t stream)
{
    // the widest two-block rings leave room for three waves per SIMD: workgroups of four waves
    // then fill a compute unit (three of them), workgroups of eight would not (one)
    constexpr int W = (V > 1 && S >= 7) ? 4 : AGC_SCALE_WAVES;
    const int64_t nblocks = (a.d + kBlockCoords - 1) / kBlockCoords;
    const int64_t per_wg = (int64_t)W * V;
    const dim3 g((unsigned)((nblocks + per_wg - 1) / per_wg)), b(kWave * W);
    if (a.full) hipLaunchKernelGGL((k_scale_pass<S, 1, W, V, true>), g, b, 0, stream, G, code.row_ptr, code.col, code.val, a);
    else hipLaunchKernelGGL((k_scale_pass<S, 1, W, V>), g, b, 0, stream, G, code.row_ptr, code.col, code.val, a);
}

template <int S>
static hipError_t launch_scale_pass_s(const float* G, const CodeDev& code, const ScaleArgs& a,
                                      int scale_mode, hipStream_t stream)
{
    if (S != kStreamDriver && code.parts && !a.full) {
        if constexpr (S == kStreamDriver) {
        } else if (scale_mode == 0)
            hipLaunchKernelGGL((k_scale_pass_parts<S, 0>), dim3((unsigned)a.nseg), dim3(kWave * kParts * kSegBlocks), 0,
                               stream, G, code.row_ptr, code.col, code.val, a);
        else
            hipLaunchKernelGGL((k_scale_pass_parts<S, 1>), dim3((unsigned)((a.d + kBlockCoords - 1) / kBlockCoords)),
                               dim3(kWave * kParts), 0, stream, G, code.row_ptr, code.col, code.val, a);
        return hipGetLastError();
    }
    if (scale_mode == 0) {
        hipLaunchKernelGGL((k_scale_pass<S, 0, kSegBlocks, 1>), dim3((unsigned)a.nseg), dim3(kWgThreads), 0, stream, G,
                           code.row_ptr, code.col, code.val, a);
    } else {
        // two blocks per wave where a ring driver serves the code and the vector is long enough
        // to fill the chip with half as many waves
        const int64_t nblocks = (a.d + kBlockCoords - 1) / kBlockCoords;
        if (S != 0 && AGC_SCALE_BLOCKS_PER_WAVE > 1 && nblocks >= kTwoBlockMin) launch_scale_max<S, AGC_SCALE_BLOCKS_PER_WAVE>(G, code, a, stream);
        else launch_scale_max<S, 1>(G, code, a, stream);
    }
    return hipGetLastError();
}

hipError_t launch_scale_pass(const float* G, int64_t ldg, int n, int k, int64_t d,
                             const CodeDev& code, int scale_mode, const Workspace& ws,
                             const SketchDev* sk, hipStream_t stream)
{
    const bool layers = ws.n_layers > 0;
    ScaleArgs a{ldg, n, k, d, layers && scale_mode == 0 ? ws.nseg_layers : ws.nseg, ws.part_max, ws.part_sq, code.win, code.stream,
                layers && scale_mode == 1 ? ws.block_layer : nullptr,
                layers && scale_mode == 0 ? ws.seg_first : nullptr, layers && scale_mode == 0 ? ws.seg_blocks : nullptr, sk ? sk->state + 2 : nullptr, sk ? sk->limit : 0u};
    if (code.band < 0 && !code.win) return hipErrorInvalidValue;  // the window driver reads the records
    switch (code.band) {
        case 1: return launch_scale_pass_s<1>(G, code, a, scale_mode, stream);
        case 2: return launch_scale_pass_s<2>(G, code, a, scale_mode, stream);
        case 3: return launch_scale_pass_s<3>(G, code, a, scale_mode, stream);
        case 4: return launch_scale_pass_s<4>(G, code, a, scale_mode, stream);
        case 5: return launch_scale_pass_s<5>(G, code, a, scale_mode, stream);
        case 6: return launch_scale_pass_s<6>(G, code, a, scale_mode, stream);
        case 7: return launch_scale_pass_s<7>(G, code, a, scale_mode, stream);
        case 8: return launch_scale_pass_s<8>(G, code, a, scale_mode, stream);
        case -2: return launch_scale_pass_s<-2>(G, code, a, scale_mode, stream);
        case -4: return launch_scale_pass_s<-4>(G, code, a, scale_mode, stream);
        case -8: return launch_scale_pass_s<-8>(G, code, a, scale_mode, stream);
        default:
            return code.stream && (sk || !code.parts) ? launch_scale_pass_s<kStreamDriver>(G, code, a, scale_mode, stream)
                                              : launch_scale_pass_s<0>(G, code, a, scale_mode, stream);
    }
}

// =======================================================================================
// K1f  scale finalize: one workgroup per worker
// =======================================================================================
// acc = acc + rows b0, b0 + 1, .. of part, BATCH of them or up to s1; past s1 the last row is read again
template <int BATCH>
__device__ __forceinline__ void add_rows(const double* part, int n, int64_t b0, int64_t s1, double& acc)
{
    double v[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = part[(b0 + u < s1 ? b0 + u : s1 - 1) * n];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) acc = b0 + u < s1 ? acc + v[u] : acc;
}

// Euclidean scale, level 3 of the tree: one workgroup per group of up to 64 segments, thread t follows
// worker t through the group's rows of [segment][worker] (coalesced) and adds them in segment order.  The
// rows are requested 32 at a time before the first addition: the kernel is one round trip to memory per
// batch (batches of eight took 7-9 us, mostly waiting; now 5-6); the last eight or fewer are a batch of eight
// (of 32, where 28 additions are thrown away, one to three workers x 4096 were 1 us slower).  With layer-wise scales the groups of
// every layer are counted from its first segment and listed in group_seg.
__global__ __launch_bounds__(kWgThreads) void k_scale_groups(int n, Workspace ws, int64_t ngroup)
{
    const int64_t g = blockIdx.x;
    int64_t s0 = g * kGroupSegs, s1 = s0 + kGroupSegs < ws.nseg ? s0 + kGroupSegs : ws.nseg;
    if (ws.n_layers > 0) {
        s0 = ws.group_seg[g];
        s1 = ws.group_seg[g + 1];
    }
    for (int i = threadIdx.x; i < n; i += kWgThreads) {
        const double* part = ws.part_sq + i;
        double acc = 0.0;
        int64_t b0 = s0;
        for (; s1 - b0 > 8; b0 += 32) add_rows<32>(part, n, b0, s1, acc);
        if (b0 < s1) add_rows<8>(part, n, b0, s1, acc);
        ws.group_sq[(int64_t)i * ngroup + g] = acc;
    }
}

// record of one worker for the quantize pass
template <int CAP>
__device__ __forceinline__ WorkerQ worker_record(const QuantList<CAP>& in, int i, int n, float inv, float coef)
{
    // the staging area is written out after the last worker and before every worker that starts a new fill
    const uint32_t flush = (i == n - 1 || in.stage_start[i + 1] == 0) ? 1u : 0u;
    return WorkerQ{inv, (uint32_t)in.bits[i], in.codes[i], in.fuse ? coef : 0.f, in.fuse ? (uint32_t)in.arrived[i] : 0u,
                   8u * in.stage_start[i], flush};
}

// decode weight of one grid unit, as the decode prologue forms it
__device__ __forceinline__ float unit_weight(float w, float scale, int b)
{
    const double L = b >= 2 ? (double)((1 << (b - 1)) - 1) : 1.0;
    return (float)(((double)w * (double)scale) / L);
}

// What the finalize kernel needs behind a sketch: what it checks, and the places of k_resolve.  Arguments of these instances alone,
// since the host pays by the byte.
template <int CAP, bool SK>
struct SketchSide {
    const float* lo_scale;  // Euclidean: the lower bounds that it was made with
    uint32_t* state;
    uint4* table;           // k_resolve's
    uint32_t limit;         // largest magnitude: with state[2] above this there is no sketch
    uint16_t start[CAP];    // stage_starts() of the fills of k_resolve
};
template <int CAP>
struct SketchSide<CAP, false> {};
template <int CAP>
static SketchSide<CAP, true> sketch_side(int n, const SketchDev& sk, const QuantStreams& out)
{
    SketchSide<CAP, true> side{sk.lo_scale, sk.state, sk.table, sk.limit, {}};
    for (int i = 0; i < n; ++i) side.start[i] = out.resolve_start[i];
    return side;
}

// One workgroup per worker (and layer, with the Euclidean scale).  SK: behind a sketch; with the places of k_resolve found here, from the
// widths of the workers before, the kernel took 5.96 us instead of 4.72 (64 workers x 1 M, Euclidean).
template <int MODE, int CAP, bool SK>
__global__ __launch_bounds__(kWgThreads) void k_scale_finalize(int n, QuantList<CAP> in, Workspace ws, int64_t ngroup,
                                                               SketchSide<CAP, SK> side, float* scales)
{
    const int i = blockIdx.x;
    const int tid = threadIdx.x;
    float scale;
    uint32_t cost = 0u;  // of the sampled blocks
    if constexpr (SK && MODE == 1) {
        if (i == 0 && tid == 0) cost = side.state[2];
    }
    if (MODE == 1) {
        __shared__ uint32_t red[kWgThreads];
        // this worker's column of the slot array: read it with loads that see the atomics of the
        // scale pass (they were performed in memory, past the caches), and leave zeros behind
        uint32_t m = 0u;
        for (int sl = tid; sl < kMaxSlots; sl += kWgThreads) {
            uint32_t* p = ws.part_max + (int64_t)sl * n + i;
            m = max(m, __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            __hip_atomic_store(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        red[tid] = m;
        __syncthreads();
        for (int h = kWgThreads / 2; h > 0; h >>= 1) {
            if (tid < h) red[tid] = max(red[tid], red[tid + h]);
            __syncthreads();
        }
        scale = __uint_as_float(red[0]);
    } else {
        // Level 3 (64 segments -> group) was formed by k_scale_groups.  Four supergroups at a time: one
        // thread per group fetches it, one per supergroup adds its 64 groups in order (level 4), the first
        // adds the supergroups in order (level 5).
        __shared__ double group[kWgThreads];
        __shared__ double super[kWgThreads / kGroupSegs];
        const int64_t g_begin = ws.n_layers > 0 ? ws.layer_group[blockIdx.y] : 0;
        const int64_t g_end = ws.n_layers > 0 ? ws.layer_group[blockIdx.y + 1] : ngroup;
        const double* sq = ws.group_sq + (int64_t)i * ngroup;
        double total = 0.0;
        for (int64_t g0 = g_begin; g0 < g_end; g0 += kWgThreads) {
            if (g0 + tid < g_end) group[tid] = sq[g0 + tid];
            __syncthreads();
            if (tid < kWgThreads / kGroupSegs) {
                const int64_t left = g_end - g0 - tid * kGroupSegs;
                const int have = left < kGroupSegs ? (int)left : kGroupSegs;
                double acc = 0.0;
                for (int u = 0; u < have; ++u) acc = acc + group[tid * kGroupSegs + u];
                super[tid] = acc;
            }
            __syncthreads();
            if (tid == 0)
                for (int u = 0; u < kWgThreads / kGroupSegs && g0 + u * kGroupSegs < g_end; ++u) total = total + super[u];
        }
        scale = (float)sqrt(total);  // thread 0 holds the total, and it alone goes on
    }
    if (tid == 0) {
        const int l = MODE == 0 ? (int)blockIdx.y : 0, per = MODE == 0 ? (int)gridDim.y : 1;
        scales[(int64_t)i * per + l] = scale;
        const int b = in.bits[i];
        const WorkerQ q = worker_record(in, i, n, inv16_of(scale, b), unit_weight(in.w[i], scale, b));
        ws.wq[(int64_t)l * n + i] = q;
        if constexpr (SK) {
            const uint32_t ends = i == n - 1 || side.start[i + 1] == 0 ? 512u : 0u;
            side.table[i] = make_uint4(__float_as_uint(q.inv16), __float_as_uint(q.coef), q.bits | (q.arrived << 8) | ends,
                                       32u * side.start[i]);
            if (MODE == 1 && i == 0) side.state[2] = 0u;  // the next step's
            bool made = true;
            if constexpr (MODE == 1) made = cost <= side.limit;
            else made = scale >= side.lo_scale[i];
            // a weight that is not finite makes NaN of zero levels too, which k_resolve does not add up
            if (!(made && fabsf(q.coef) < __builtin_inff()))
                (void)__hip_atomic_fetch_or(side.state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Layer-wise largest-magnitude scales: workgroup l, thread i.  The kLayerSub rows of layer l in the slot
// array hold the layer's maxima; every (worker, layer) gets its scale, and table l of the quantize pass gets
// the worker's record with the multiplier and the decode weight of that layer (the formulas of the
// per-vector case with the layer's scale).  The rows are handed back zeroed.
template <int CAP>
__global__ __launch_bounds__(kWgThreads) void k_scale_finalize_layers(int n, QuantList<CAP> in, Workspace ws, float* scales)
{
    const int l = blockIdx.x;
    for (int i = threadIdx.x; i < n; i += kWgThreads) {
        uint32_t m = 0u;
        for (int r = 0; r < kLayerSub; ++r) {
            uint32_t* p = ws.part_max + ((int64_t)l * kLayerSub + r) * n + i;
            m = max(m, __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            __hip_atomic_store(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const float scale = __uint_as_float(m);
        scales[(int64_t)i * ws.n_layers + l] = scale;
        const int b = in.bits[i];
        ws.wq[(int64_t)l * n + i] = worker_record(in, i, n, inv16_of(scale, b), unit_weight(in.w[i], scale, b));
    }
}

// the per-worker arguments of the table kernels, as large as n needs
template <int CAP>
static QuantList<CAP> quant_list(int n, const QuantStreams& out, const StepWeights& sw)
{
    QuantList<CAP> q;
    q.fuse = sw.fuse;
    for (int i = 0; i < n; ++i) {
        q.codes[i] = out.codes[i];
        q.bits[i] = out.bits[i];
        q.stage_start[i] = out.stage_start[i];
        q.w[i] = sw.fuse ? sw.w[i] : 0.f;
        q.arrived[i] = sw.fuse ? sw.arrived[i] : (uint8_t)0;
    }
    return q;
}

template <int CAP>
static hipError_t launch_scale_finalize_cap(int n, int scale_mode, const QuantStreams& out, const StepWeights& sw,
                                            const Workspace& ws, const SketchDev* sk, float* scales, hipStream_t stream)
{
    const QuantList<CAP> q = quant_list<CAP>(n, out, sw);
    const int layers = ws.n_layers;
    if (scale_mode == 1) {
        if (layers > 0)
            hipLaunchKernelGGL((k_scale_finalize_layers<CAP>), dim3(layers), dim3(kWgThreads), 0, stream, n, q, ws, scales);
        else {
            if (sk) hipLaunchKernelGGL((k_scale_finalize<1, CAP, true>), dim3(n), dim3(kWgThreads), 0, stream, n, q, ws, (int64_t)0, sketch_side<CAP>(n, *sk, out), scales);
            else hipLaunchKernelGGL((k_scale_finalize<1, CAP, false>), dim3(n), dim3(kWgThreads), 0, stream, n, q, ws, (int64_t)0, SketchSide<CAP, false>{}, scales);
        }
        return hipGetLastError();
    }
    const int64_t ngroup = layers > 0 ? ws.ngroup_layers : ws.ngroup;
    hipLaunchKernelGGL(k_scale_groups, dim3((unsigned)ngroup), dim3(kWgThreads), 0, stream, n, ws, ngroup);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 g(n, layers > 0 ? layers : 1), b(kWgThreads);
    if (sk) hipLaunchKernelGGL((k_scale_finalize<0, CAP, true>), g, b, 0, stream, n, q, ws, ngroup, sketch_side<CAP>(n, *sk, out), scales);
    else hipLaunchKernelGGL((k_scale_finalize<0, CAP, false>), g, b, 0, stream, n, q, ws, ngroup, SketchSide<CAP, false>{}, scales);
    return hipGetLastError();
}

// The host pays about 1.7 ns per byte of kernel arguments (64 bytes 2.5 us a launch, 4000 bytes 9.1 us), so the
// lists come in three sizes.
hipError_t launch_scale_finalize(int n, int scale_mode, const QuantStreams& out, const StepWeights& sw,
                                 const Workspace& ws, const SketchDev* sk, float* scales, hipStream_t stream)
{
    if (n <= 16) return launch_scale_finalize_cap<16>(n, scale_mode, out, sw, ws, sk, scales, stream);
    if (n <= 64) return launch_scale_finalize_cap<64>(n, scale_mode, out, sw, ws, sk, scales, stream);
    return launch_scale_finalize_cap<kArgWorkers>(n, scale_mode, out, sw, ws, sk, scales, stream);
}

// ---- lower bounds of the Euclidean scales from a sample of the blocks (agc_sketch.h).  The sample's sum of squares
// without its two largest blocks, scaled up to the vector, estimates the square of the scale from below; the bound is 0.7 of
// its root.  A coordinate becomes a record with a probability in proportion to scale / bound, so a lower bound
// costs records; a higher one costs the whole sketch when the scale falls below it.  With heavy tails (Student's t, three
// degrees) one block in a sample of 131072 coordinates that holds an extreme value put the plain estimate 40 % too high in
// about 5 % of the steps of 64 workers; without the two largest blocks the bounds of 35 200 simulated workers lay at
// 0.77 of the scale at most.  Where one block in 64 holds nearly all of the norm the bound fails in 0.4 % of the
// steps with 128 samples, 0.3 % with 256 and 0.05 % with 512 (binomial counts).
constexpr int kSampleWaves = 16;  // waves that share a block: its latency is what counts
constexpr int kSampleRows = 128;  // rows of a block that 160 KB of LDS have room for

// A worker's combination from rows in LDS, [k][lane]
__device__ __forceinline__ float4 encode_staged_one(const float4* rows, const CsrView& B, int i, int lane)
{
    const int e0 = B.row_ptr[i], e1 = B.row_ptr[i + 1];
    float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int e = e0; e < e1; ++e) f = fma4(B.val[e], rows[B.col[e] * kWave + lane], f);
    return f;
}

// all rows of a block into LDS, requested together
__device__ __forceinline__ void stage_rows(const float* __restrict__ G, int64_t ldg, int k, const LaneCoords& lc, int wave, int lane,
                                           float4* rows)
{
    for (int j0 = wave; j0 < k; j0 += 4 * kSampleWaves) {
        float4 r[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int j = j0 + t * kSampleWaves;
            r[t] = load_row4<true>(G + (int64_t)(j < k ? j : k - 1) * ldg, lc);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int j = j0 + t * kSampleWaves;
            if (j < k) rows[j * kWave + lane] = r[t];
        }
    }
    __syncthreads();
}

// What the sample keeps of a block and worker for the largest-magnitude scale: the largest magnitude and the sum of all
struct EpiTopSum {
    typedef float2 Part;
    typedef float Sum;
    static constexpr bool kStoresPerWorker = false;
    static constexpr bool kWantsZeros = true;
    static constexpr int kPrefetchRows = AGC_SCALE_PREFETCH_ROWS;
    float2* acc;
    int lane;
    template <bool EVEN>
    __device__ __forceinline__ void worker(int i, const float4& f)
    {
        const uint32_t m = wave_max_nonneg_bits(EpiMaxAbs::max_abs4(f));
        float s = (fabsf(f.x) + fabsf(f.y)) + (fabsf(f.z) + fabsf(f.w));
        s += __uint_as_float(dpp_u32<kDppQuadSwap1>(__float_as_uint(s)));
        s += __uint_as_float(dpp_u32<kDppQuadSwap2>(__float_as_uint(s)));
        s += __uint_as_float(dpp_u32<kDppHalfMirror>(__float_as_uint(s)));
        s += __uint_as_float(dpp_u32<kDppRowMirror>(__float_as_uint(s)));
        const uint32_t v = __float_as_uint(s);
        s = (__uint_as_float(__builtin_amdgcn_readlane(v, 0)) + __uint_as_float(__builtin_amdgcn_readlane(v, 16))) +
            (__uint_as_float(__builtin_amdgcn_readlane(v, 32)) + __uint_as_float(__builtin_amdgcn_readlane(v, 48)));
        if (lane == 0) acc[i] = make_float2(__uint_as_float(m), s);
    }
    __device__ __forceinline__ void worker_any(int i, const float4& f) { worker<true>(i, f); }
};

constexpr int kBoundRows = 16;  // rows of the array of running maxima that the sample is folded into

// What bounds it: latency, one block per workgroup and all workgroups resident at once.  S > 0: the register ring.  Other codes
// with STAGED: all rows of the block are requested at once and wait in LDS, where each wave takes its workers' from; else
// rows are gathered from memory (more rows than LDS holds).  64 workers x 25.6 M, window of 8: the window driver, whose
// unrolled code comes cold into the instruction cache, took 20.9 us, with 4 | 8 | 12 rows requested ahead 19.6 | 38.9 |
// 39.0, staged 11.2;  50 x 5.4 M 19.9 | 8.4;  10 workers of 30 partitions, gathered 8.4, staged 5.9.  The ring of a cyclic band
// is the faster one: 64 x 1 M 5.6, staged 7.1, 32 x 11.7 M 6.2 and 8.0.  Code entries one a lane instead of scalar loads,
// a worker ahead: 13.2 for 11.2.
//
// sums: [sample][worker], sums of squares or of magnitudes; maxima go to the first rows of a.part_max
template <int S, bool STAGED, class Epi>
__global__ __launch_bounds__(kWave * kSampleWaves) void k_sketch_sample(const float* __restrict__ G, const int* __restrict__ row_ptr,
                                                                        const int* __restrict__ col, const float* __restrict__ val,
                                                                        ScaleArgs a, SampleRuns runs, typename Epi::Sum* sums)
{
    extern __shared__ __attribute__((aligned(16))) float4 lds_rows[];  // STAGED: [k][64]
    __shared__ typename Epi::Part lds_part[kMaxWorkers];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t base = sample_block(runs, blockIdx.x) * kBlockCoords;
    const LaneCoords lc = lane_coords(base, lane, a.d);
    const CsrView B{row_ptr, col, val, nullptr};
    Epi epi{lds_part, lane};
    auto hand_in = [&](int i) {
        if constexpr (std::is_same<Epi, EpiTopSum>::value) {
            (void)__hip_atomic_fetch_max(a.part_max + (blockIdx.x % kBoundRows) * a.n + i, __float_as_uint(lds_part[i].x),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sums[(int64_t)blockIdx.x * a.n + i] = lds_part[i].y;
        } else {
            sums[(int64_t)blockIdx.x * a.n + i] = lds_part[i];
        }
    };
    if constexpr (S > 0) {
        const int size = ((a.n + kSampleWaves - 1) / kSampleWaves + 1) / 2 * 2;
        const int i0 = wave * size, i1 = i0 + size < a.n ? i0 + size : a.n;
        encode_block_part<S>(G + base, a.ldg, a.k, B, lc, i0, i1, epi);
        for (int i = i0 + lane; i < i1; i += kWave) hand_in(i);  // of this wave's lane 0
        return;
    }
    if constexpr (STAGED) {
        stage_rows(G + base, a.ldg, a.k, lc, wave, lane, lds_rows);
    }
    for (int i = wave; i < a.n; i += kSampleWaves) {
        const float4 f = STAGED ? encode_staged_one(lds_rows, B, i, lane) : encode_gather_one(G + base, a.ldg, B, i, lc);
        epi.template worker<true>(i, valid_coords(f, lc.nvalid));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < a.n; i += kWave * kSampleWaves) hand_in(i);
}

__global__ __launch_bounds__(kWgThreads) void k_sketch_bounds(int n, BitList in, const double* part_sq, int samples,
                                                              double times, SketchDev sk)
{
    __shared__ double sum[kWgThreads], top[kWgThreads], second[kWgThreads];
    const int i = blockIdx.x, tid = threadIdx.x;
    double s = 0.0, m1 = 0.0, m2 = 0.0;
    for (int e = tid; e < samples; e += kWgThreads) {
        const double v = part_sq[(int64_t)e * n + i];
        s = s + v;
        m2 = fmax(m2, fmin(m1, v));
        m1 = fmax(m1, v);
    }
    sum[tid] = s;
    top[tid] = m1;
    second[tid] = m2;
    __syncthreads();
    for (int h = kWgThreads / 2; h > 0; h >>= 1) {
        if (tid < h) {
            sum[tid] = sum[tid] + sum[tid + h];
            second[tid] = fmax(fmax(second[tid], second[tid + h]), fmin(top[tid], top[tid + h]));
            top[tid] = fmax(top[tid], top[tid + h]);
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double rest = sum[0] - (samples >= 8 ? top[0] + second[0] : 0.0);
        const float lo = (float)(0.7 * sqrt(fmax(rest, 0.0) * times));
        const float mult = inv16_of(lo, in.bits[i]);
        sk.lo_scale[i] = lo;
        sk.lo_mult[i] = mult > 0.f ? mult : __builtin_inff();  // no bound, or a quotient beyond binary32
        if (i == 0) sk.state[0] = sk.state[1] = 0u;
    }
}

// The same for the largest-magnitude scale, whose bounds always hold, and whether the sketch is worth making: what the sampled
// blocks would cost, in parts of a second read of their rows (sketch_max_limit).  A coordinate becomes a record with a
// probability of L |f| / bound.  The bounds rise as k_sketch_max goes on where the values have tails, which the sample shows: how far
// the largest magnitude of all of it lies above the mean of those of its sixteenths.  Values of bounded size have 1,
// Gaussian ones 1.1, heavy tails (t, three degrees) about 1.8.  Once more for every further factor of sixteen gives
// the average block's bounds (heavy tails: three and more times those of the sample), from which follows what records cost;  whether a block
// fits is asked with half as much again at most, since the first blocks find the sample's bounds, and one standard deviation of
// room left.  The bounds go to the first row of the array of running maxima.
constexpr int kBoundsWgs = 16;
constexpr int kBoundsThreads = 1024;
__global__ __launch_bounds__(kBoundsThreads) void k_sketch_bounds_max(int n, BitList in, const float* __restrict__ sums, int samples,
                                                                      float sixteens, uint32_t* part_max, SketchDev sk)
{
    __shared__ float2 per_sum[kMaxWorkers];  // expected records for each of a block's sum of magnitudes: early, average
    __shared__ uint32_t lds_cost;            // one addition to memory a workgroup: one a wave took 3 us
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    if (tid == 0) lds_cost = 0u;
    if (tid < n) {
        uint32_t m[kBoundRows];
        float parts = 0.f;  // without the first row, which the first workgroup is raising
#pragma unroll
        for (int t = 0; t < kBoundRows; ++t) m[t] = __hip_atomic_load(part_max + t * n + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int t = 1; t < kBoundRows; ++t) {
            parts += __uint_as_float(m[t]);
            m[0] = max(m[0], m[t]);
        }
        // the chip's own reciprocal, logarithm and exponential: a decision, no result
        const float top = __uint_as_float(m[0]);
        const float rise = fmaxf((float)(kBoundRows - 1) * top * __builtin_amdgcn_rcpf(parts), 1.f);  // 1 where that is not a number
        const float per = m[0] != 0u ? (float)((1 << (in.bits[tid] - 1)) - 1) * __builtin_amdgcn_rcpf(top) : 0.f;
        per_sum[tid] = make_float2(per * __builtin_amdgcn_rcpf(fminf(rise, 1.5f)),
                                   per * __builtin_amdgcn_rcpf(fminf(__builtin_amdgcn_exp2f(sixteens * __builtin_amdgcn_logf(rise)), 3.f)));
        if (blockIdx.x == 0) (void)__hip_atomic_fetch_max(part_max + tid, m[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const float room = (float)sk.cap, most = room - sqrtf(room), unit = 0.5f * kReadCost / room;
    uint32_t cost = 0u;
    for (int e = blockIdx.x + wave * kBoundsWgs; e < samples; e += kBoundsWgs * (kBoundsThreads / kWave)) {
        float early = 0.f, average = 0.f;
        for (int j = lane; j < n; j += kWave) {
            const float sum = sums[(int64_t)e * n + j];
            const float r = sum * per_sum[j].x, q = sum * per_sum[j].y;
            early += r < (float)kBlockCoords ? r : (float)kBlockCoords;
            average += q < (float)kBlockCoords ? q : (float)kBlockCoords;
        }
#pragma unroll
        for (int h = 1; h < kWave; h *= 2) {
            early += __shfl_xor(early, h);
            average += __shfl_xor(average, h);
        }
        cost += early > most ? kReadCost : (uint32_t)(unit * fminf(average, room));
    }
    if (lane == 0) atomicAdd(&lds_cost, cost);
    __syncthreads();
    if (tid == 0 && lds_cost != 0u) (void)__hip_atomic_fetch_add(sk.state + 2, lds_cost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (blockIdx.x == 0 && tid == 0) sk.state[0] = sk.state[1] = 0u;
}

template <int S, bool STAGED, class Epi>
static void launch_sketch_sample_s(const float* G, const CodeDev& code, const ScaleArgs& a, int samples, const SampleRuns& runs,
                                   typename Epi::Sum* sums, hipStream_t stream)
{
    hipLaunchKernelGGL((k_sketch_sample<S, STAGED, Epi>), dim3(samples), dim3(kWave * kSampleWaves),
                       STAGED ? sizeof(float4) * kWave * a.k : 0, stream, G, code.row_ptr, code.col, code.val, a, runs, sums);
}

template <class Epi>
static hipError_t launch_sketch_sample(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code, int samples,
                                       uint64_t seed, uint64_t step, uint32_t* part_max, typename Epi::Sum* sums, hipStream_t stream)
{
    const SampleRuns runs = sample_runs((d + kBlockCoords - 1) / kBlockCoords, samples, seed, step);
    const ScaleArgs a{ldg, n, k, d, 0, part_max, nullptr, code.win, nullptr, nullptr, nullptr, nullptr, nullptr, 0u};
    switch (code.band) {
        case 1: launch_sketch_sample_s<1, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 2: launch_sketch_sample_s<2, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 3: launch_sketch_sample_s<3, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 4: launch_sketch_sample_s<4, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 5: launch_sketch_sample_s<5, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 6: launch_sketch_sample_s<6, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 7: launch_sketch_sample_s<7, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        case 8: launch_sketch_sample_s<8, false, Epi>(G, code, a, samples, runs, sums, stream); break;
        default:
            if (k <= kSampleRows) launch_sketch_sample_s<0, true, Epi>(G, code, a, samples, runs, sums, stream);
            else launch_sketch_sample_s<0, false, Epi>(G, code, a, samples, runs, sums, stream);
    }
    return hipGetLastError();
}

hipError_t launch_sketch_bounds(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code,
                                const Workspace& ws, const SketchDev& sk, const QuantStreams& out, uint64_t seed,
                                uint64_t step, hipStream_t stream)
{
    // the partial sums' array is their scratch, which has a row for every four blocks
    const int64_t nblocks = (d + kBlockCoords - 1) / kBlockCoords;
    const int samples = sample_count(nblocks);
    const hipError_t e = launch_sketch_sample<EpiSumSq>(G, ldg, n, k, d, code, samples, seed, step, nullptr, ws.part_sq, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sketch_bounds, dim3(n), dim3(kWgThreads), 0, stream, n, bit_list(n, out), ws.part_sq, samples,
                       (double)nblocks / (double)samples, sk);
    return hipGetLastError();
}

hipError_t launch_sketch_bounds_max(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code,
                                    const Workspace& ws, const SketchDev& sk, const QuantStreams& out, uint64_t seed,
                                    uint64_t step, hipStream_t stream)
{
    // the records' array is scratch: four bytes for a worker and sample, of which there are no more than blocks, in a room of
    // at least 2048 bytes a block (256 records)
    const int samples = sample_count((d + kBlockCoords - 1) / kBlockCoords);
    float* sums = reinterpret_cast<float*>(sk.recs);
    const hipError_t e = launch_sketch_sample<EpiTopSum>(G, ldg, n, k, d, code, samples, seed, step, ws.part_max, sums, stream);
    if (e != hipSuccess) return e;
    const float sixteens = (float)(log2((double)((d + kBlockCoords - 1) / kBlockCoords) / samples) / log2((double)kBoundRows));
    hipLaunchKernelGGL(k_sketch_bounds_max, dim3(kBoundsWgs), dim3(kBoundsThreads), 0, stream, n, bit_list(n, out), sums, samples, sixteens,
                       ws.part_max, sk);
    return hipGetLastError();
}

// =======================================================================================
// K2  encode + stochastic quantize + bit-pack: kernels in agc_quantize.h, instantiated in
// agc_quantize_b0/b1/b2.hip; here the table prologue and the launch entry points
// =======================================================================================
// table of the bucket-wise pass: bit-width and stream of every worker (the multiplier is
// found per block inside the pass)
template <int CAP>
__global__ __launch_bounds__(kWgThreads) void k_quant_table(int n, QuantList<CAP> in, WorkerQ* wq)
{
    const int i = threadIdx.x;
    if (i >= n) return;
    const int b = in.bits[i];
    // bucket-wise scales: the multiplier is num / scale with the block's own scale; the record
    // carries the numerator L * 2^16 (2^15 for a one-bit worker)
    const float num = b >= 2 ? (float)(((1u << (b - 1)) - 1u) << 16) : 32768.0f;
    const double L = b >= 2 ? (double)((1 << (b - 1)) - 1) : 1.0;
    wq[i] = worker_record(in, i, n, num, (float)((double)in.w[i] / L));
}

hipError_t launch_quantize_bucket(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code,
                                  int scale_mode, const QuantStreams& out, const StepWeights& sw,
                                  const Workspace& ws, float* scales, uint64_t seed, uint64_t step, float* ghat,
                                  hipStream_t stream)
{
    if (n <= 16)
        hipLaunchKernelGGL(k_quant_table<16>, dim3(1), dim3(kWgThreads), 0, stream, n, quant_list<16>(n, out, sw), ws.wq);
    else if (n <= 64)
        hipLaunchKernelGGL(k_quant_table<64>, dim3(1), dim3(kWgThreads), 0, stream, n, quant_list<64>(n, out, sw), ws.wq);
    else
        hipLaunchKernelGGL(k_quant_table<kArgWorkers>, dim3(1), dim3(kWgThreads), 0, stream, n,
                           quant_list<kArgWorkers>(n, out, sw), ws.wq);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    QuantArgs a{ldg, n, k, d, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32),
                scales, (d + kBlockCoords - 1) / kBlockCoords, ghat, nullptr, nullptr, out.stage_bits, out.stage_fills,
                nullptr, 0u, out.parts, nullptr, nullptr};
    if (a.stage_fills > 1)
        return scale_mode == 0 ? launch_quantize_band2m(G, code, ws, a, stream)
                               : launch_quantize_band1m(G, code, ws, a, stream);
    return scale_mode == 0 ? launch_quantize_band2s(G, code, ws, a, stream)
                           : launch_quantize_band1s(G, code, ws, a, stream);
}

hipError_t launch_quantize(const float* G, int64_t ldg, int n, int k, int64_t d,
                           const CodeDev& code, const Workspace& ws, const QuantStreams& out, uint64_t seed,
                           uint64_t step, float* ghat, const SketchDev* sk, hipStream_t stream)
{
    QuantArgs a{ldg, n, k, d, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32),
                nullptr, 0, ghat, nullptr, nullptr, out.stage_bits, out.stage_fills,
                ws.n_layers > 0 ? ws.block_layer : nullptr, 0u, out.parts, sk ? sk->state : nullptr, sk ? sk->left : nullptr};
    return a.stage_fills > 1 ? launch_quantize_band0m(G, code, ws, a, stream)
                             : launch_quantize_band0s(G, code, ws, a, stream);
}

// =======================================================================================
// K3  masked dequantize + weighted sum
// =======================================================================================
// A workgroup takes tiles of 256 * COORDS coordinates (a lane owns COORDS consecutive ones) and walks, in
// every tile, over the arrived workers in ascending order.  A b-bit worker's part of a tile is b "units"
// of 32 * COORDS contiguous bytes of its stream; the units of consecutive workers are packed into chunks
// of 12 KB.  All lanes fetch a chunk together, three 16-byte pieces each, wholly coalesced
// and without a branch, into registers while the chunk before it is decoded from LDS, also across the end
// of a tile.
//
// What bounds it: instruction issue.  At the metric size (25.6 M coordinates, 43 of 64 workers arrived) a
// wave spends about 70 vector and 28 scalar instructions on 16 codes of each lane: 7.6e7 vector instructions
// in 0.14 ms, 0.86 of one in four clocks on every SIMD; the memory would allow 0.09 ms.  The first form of the
// kernel let every lane load its own b words of one worker right before they were used and decode 32 codes of
// them: one request in flight per wave, 0.169 ms, and 26 us even for 200 000 coordinates (20 workers times one
// round trip to memory).  This form: 0.148 ms and 18 us with resident workgroups that walk over the tiles,
// 0.137-0.143 ms with one workgroup per tile (decode_groups).  Six waves per SIMD (72 vector registers, 24 KB of
// LDS), walking: five take 0.162 ms, four with chunks of 16 KB 0.166 ms, eight with 8 KB 0.160 ms.
constexpr int kDecPieces = kDecChunkBytes / 16;            // 16-byte pieces of a chunk
constexpr int kDecPerThread = kDecPieces / kWgThreads;
static_assert(kDecPerThread * kWgThreads == kDecPieces, "every lane fetches the same number of pieces");
constexpr int kDecAux = 512;                               // (workers of a chunk) x (buckets of a tile), at most

// true when x / 2 is exact in binary32: zero, or a normal number that stays normal
__device__ __forceinline__ bool halves_exactly(float x)
{
    const uint32_t u = __float_as_uint(x), e = (u >> 23) & 0xFFu;
    return ((u << 1) == 0u) | (e - 2u < 0xFDu);
}

// One workgroup per layer (one in all without layer-wise scales); the first also writes the tables of
// streams: one record per arrived worker, one per unit, and the first worker of every chunk.
// SCALES 0: one scale per worker, folded into the weight here.  1: bucket-wise; the record holds w_i / L_i
// and the product with the bucket's scale is formed in the decode.  2: layer-wise; the weights go to
// [layer][slot].
template <int CAP, int SCALES, bool TWO>
__global__ __launch_bounds__(kWgThreads) void k_decode_table(DecodeList<CAP> in, const float* scales, int n_layers,
                                                             DecodeTables tab, float* coef_layer, float* coef2_layer)
{
    const int i = threadIdx.x;
    const int l = blockIdx.x;
    const int n = in.n_arrived;
    const int per_chunk = in.units_per_chunk;
    auto write_unit = [&](int of, int u) {  // slot u of the chunk of worker `of`
        const int bits = in.bits[of], mine = u - in.pos[of];
        const uint32_t pieces = in.groups * (uint32_t)bits;  // of the whole stream
        uint32_t at = (uint32_t)((mine < bits ? mine : bits - 1) * in.unit_pieces);
        if (at >= pieces) at = 0;  // a unit past the end of a short stream: nobody uses what is read
        tab.units[(int64_t)in.chunk[of] * per_chunk + u] =
            DecUnit{(const char*)in.codes[of] + (int64_t)at * 16, (uint32_t)(bits * in.unit_pieces), pieces - at};
    };
    // The last worker of a chunk repeats its last unit up to the chunk's end (a second request of the same lines),
    // so that every piece of a chunk can be requested without a test.  In the last chunk that may be nearly all of
    // it: all threads share it (one thread alone took 2 us, a quarter of a decode of one to four workers).
    if (l == 0) {
        const int u = in.pos[n - 1] + in.bits[n - 1] + i;
        if (u < per_chunk) write_unit(n - 1, u);
    }
    if (i >= n) return;
    const int b = in.bits[i];
    const int worker = in.worker[i];
    // weight of one grid unit of the worker: w_i * scale_i / L_i, binary64 then one rounding
    const double L = b >= 2 ? (double)((1 << (b - 1)) - 1) : 1.0;
    const double sc = SCALES == 0 ? (double)scales[worker] : (SCALES == 2 ? (double)scales[(int64_t)worker * n_layers + l] : 1.0);
    const float c1 = (float)(SCALES == 1 ? (double)in.w[i] / L : ((double)in.w[i] * sc) / L);
    float c2 = 0.f;
    if (TWO) c2 = (float)(SCALES == 1 ? (double)in.v[i] / L : ((double)in.v[i] * sc) / L);
    if (SCALES == 2) {
        coef_layer[(int64_t)l * n + i] = c1;
        if (TWO) coef2_layer[(int64_t)l * n + i] = c2;
        if (l != 0) return;
    }
    const int chunk = in.chunk[i], pos = in.pos[i];
    const bool halves = SCALES == 0 && b == 2 && halves_exactly(c1) && (!TWO || halves_exactly(c2));
    tab.workers[i] = DecWorker{c1, c2, halves ? 1u : 1u << b, (uint32_t)pos, (uint32_t)worker, (uint32_t)b,
                               (const char*)in.codes[i]};
    if (per_chunk == 0) return;  // decoded without chunks
    if (pos == 0) tab.chunk_first[chunk] = i;
    if (i == n - 1) tab.chunk_first[chunk + 1] = n;
    const int end = i < n - 1 && in.pos[i + 1] == 0 ? per_chunk : pos + b;
    for (int u = pos; u < end; ++u) write_unit(i, u);
}

// acc = fma(c, v, acc), in acc's own register: left to itself the compiler gives every bit-width's branch
// registers of its own and copies all accumulators back where the branches meet (32 moves per worker
// next to 96 useful instructions for a two-bit one)
__device__ __forceinline__ void fma_into(float& acc, float c, float v)
{
    asm("v_fmac_f32_e32 %0, %1, %2" : "+v"(acc) : "v"(c), "v"(v));
}

// COORDS codes of B bits, from words in which the first one starts at bit 0
template <int B, int COORDS, int NW, bool TWO>
__device__ __forceinline__ void decode_words(const uint32_t (&w)[NW], float coef, float coef2, float (&acc)[COORDS],
                                             float (&acc2)[TWO ? COORDS : 1])
{
#pragma unroll
    for (int q = 0; q < COORDS; ++q) {
        const int bit = q * B;
        const int wi = bit >> 5, sh = bit & 31;
        float v;
        if (B == 1) {
            v = __uint_as_float((~(w[wi] << (31 - sh)) & 0x80000000u) | 0x3F800000u);  // 1: +1, 0: -1
        } else {
            // the code's low B-1 bits are the level, its top bit the sign
            uint32_t x = w[wi];
            int s = sh;
            if (sh + B > 32) {  // the code straddles two words: bring it down to bit 0
                x = __builtin_amdgcn_alignbit(w[(wi + 1) < NW ? (wi + 1) : wi], w[wi], sh);
                s = 0;
            }
            const uint32_t level = (x >> s) & ((1u << (B - 1)) - 1u);
            const uint32_t sign = (x << (32 - B - s)) & 0x80000000u;
            v = __uint_as_float(__float_as_uint((float)level) | sign);
        }
        fma_into(acc[q], coef, v);
        if (TWO) fma_into(acc2[TWO ? q : 0], coef2, v);
    }
}

// Two-bit workers (sign + one level bit; most workers of a tight budget): shifted to the top of a
// word, the code's two bits are the sign and the leading exponent bit of a float, i.e. the values
// +0, +2, -0, -2 = twice the decoded value.  With half the weight the fused multiply-add has the
// same exact product and therefore the same rounded result as fma(coef, +-level, acc): three
// vector instructions per code (shift, mask, fma) instead of five.  The caller guarantees that
// halving the weights is exact (they are zero or normal numbers above the smallest exponent).
template <int COORDS, int NW, bool TWO>
__device__ __forceinline__ void decode_words_2bit(const uint32_t (&w)[NW], float half_coef, float half_coef2,
                                                  float (&acc)[COORDS], float (&acc2)[TWO ? COORDS : 1])
{
#pragma unroll
    for (int q = 0; q < COORDS; ++q) {
        const int sh = 30 - 2 * (q & 15);  // brings code q of its word to bits 31..30
        const float v2 = __uint_as_float((w[q >> 4] << sh) & 0xC0000000u);
        fma_into(acc[q], half_coef, v2);
        if (TWO) fma_into(acc2[TWO ? q : 0], half_coef2, v2);
    }
}

// a lane's COORDS codes of one worker, from the worker's part of the chunk in LDS
template <int B, int COORDS, bool TWO, bool HALVES = false>
__device__ __forceinline__ void decode_worker(const uint32_t* part, float c1, float c2, float (&acc)[COORDS],
                                              float (&acc2)[TWO ? COORDS : 1])
{
    constexpr int kBytes = COORDS / 8 * B;                                  // of one lane
    constexpr int kAway = kBytes % 4 == 0 ? 0 : (kBytes % 2 == 0 ? 2 : 3);  // furthest first byte from its word
    constexpr int NW = (kBytes + 3) / 4, NIN = (kBytes + kAway + 3) / 4;
    const uint32_t off = threadIdx.x * (uint32_t)kBytes;
    uint32_t w[NW];
    if constexpr (kBytes % 16 == 0) {
        const u32x4_t* p = reinterpret_cast<const u32x4_t*>(part) + threadIdx.x * (uint32_t)(kBytes / 16);
#pragma unroll
        for (int t = 0; t < NW; t += 4) {
            const u32x4_t v = p[t / 4];
            w[t] = v.x;
            w[t + 1] = v.y;
            w[t + 2] = v.z;
            w[t + 3] = v.w;
        }
    } else if constexpr (kBytes % 8 == 0) {
        const uint2* p = reinterpret_cast<const uint2*>(part) + threadIdx.x * (uint32_t)(kBytes / 8);
#pragma unroll
        for (int t = 0; t < NW; t += 2) {
            const uint2 v = p[t / 2];
            w[t] = v.x;
            w[t + 1] = v.y;
        }
    } else {
        const uint32_t* p = part + (off >> 2);
        uint32_t in[NIN];
#pragma unroll
        for (int t = 0; t < NIN; ++t) in[t] = p[t];
#pragma unroll
        for (int t = 0; t < NW; ++t)
            w[t] = kAway ? __builtin_amdgcn_alignbyte(in[t + 1 < NIN ? t + 1 : t], in[t], off & 3u) : in[t];
    }
    if constexpr (HALVES) decode_words_2bit<COORDS, NW, TWO>(w, 0.5f * c1, 0.5f * c2, acc, acc2);
    else decode_words<B, COORDS, NW, TWO>(w, c1, c2, acc, acc2);
}

// Wave-uniform choice among the bit-widths.  The width comes as a one-hot mask (bit b; bit 0 stands for a
// two-bit worker whose weights halve exactly): the compiler does not know that only one bit is set, so the
// tests stay one-armed ifs.  An else arm would keep the accumulators' old values alive across the other
// arm, and with them a copy of every one of them (32 moves per worker next to 96 useful instructions).
template <int LO, int HI, int COORDS, bool TWO>
__device__ __forceinline__ void decode_any(uint32_t mask, const uint32_t* part, float c1, float c2,
                                           float (&acc)[COORDS], float (&acc2)[TWO ? COORDS : 1])
{
    if (mask & (1u << LO)) decode_worker<LO == 0 ? 2 : LO, COORDS, TWO, LO == 0>(part, c1, c2, acc, acc2);
    if constexpr (LO < HI) decode_any<LO + 1, HI, COORDS, TWO>(mask, part, c1, c2, acc, acc2);
}

template <int COORDS>
__device__ __forceinline__ void store_coords(float* dst, const float (&acc)[COORDS], int64_t m0, int64_t d)
{
    if (m0 + COORDS <= d) {
#pragma unroll
        for (int q = 0; q < COORDS; q += 4)
            *reinterpret_cast<float4*>(dst + q) = make_float4(acc[q], acc[q + 1], acc[q + 2], acc[q + 3]);
    } else {
#pragma unroll
        for (int q = 0; q < COORDS; ++q)
            if (m0 + q < d) dst[q] = acc[q];
    }
}

struct DecodeArgs {
    int n_arrived;
    int n_chunks;
    int64_t d;
    int64_t n_tiles;
    float* ghat;
    float* ghat2;               // second track (two-track decode only)
    const float* scales;        // bucket-wise scales only: n x nb
    int64_t nb;
    const uint8_t* block_layer; // layer-wise scales only: the layer of every block
    const float* coef_layer;    // and the weights [layer][arrived slot]
    const float* coef2_layer;
};

// LDS of a decode workgroup: two chunks, and with bucket- or layer-wise scales the weights of their workers
template <bool TWO, int SCALES>
struct DecodeLds {
    u32x4_t chunk[2][kDecPieces + 1];   // one more: a lane may read a word past its own
    float aux[SCALES ? 2 : 1][SCALES ? kDecAux : 1];
    float aux2[SCALES == 2 && TWO ? 2 : 1][SCALES == 2 && TWO ? kDecAux : 1];
    uint8_t worker[SCALES == 1 ? kMaxWorkers : 1];
};
// SCALES 0: one scale per worker (the weight of the table).  1: bucket-wise (weight of the table
// times the bucket's scale).  2: layer-wise (the weight of the lane's layer; a lane's coordinates lie in
// one block and therefore in one layer).
template <bool TWO, int SCALES, int COORDS>
__global__ __launch_bounds__(kWgThreads)
__attribute__((amdgpu_waves_per_eu(decode_per_cu(sizeof(DecodeLds<TWO, SCALES>)), decode_per_cu(sizeof(DecodeLds<TWO, SCALES>)))))
void k_decode(const DecWorker* __restrict__ workers, const DecUnit* __restrict__ units,
              const int* __restrict__ chunk_first, DecodeArgs a)
{
    constexpr int kUnitPieces = 2 * COORDS;                  // 32 * COORDS bytes
    constexpr int kChunkUnits = kDecPieces / kUnitPieces;
    static_assert(COORDS * kChunkUnits <= kDecAux, "a worker has at least one unit");
    static_assert(kChunkUnits >= 16, "every worker fits a chunk");
    __shared__ DecodeLds<TWO, SCALES> lds;
    auto& lds_chunk = lds.chunk;
    auto& lds_aux = lds.aux;
    auto& lds_aux2 = lds.aux2;
    const int tid = threadIdx.x;
    float acc[COORDS];
    float acc2[TWO ? COORDS : 1];
#pragma unroll
    for (int q = 0; q < COORDS; ++q) acc[q] = 0.f;
#pragma unroll
    for (int q = 0; q < (TWO ? COORDS : 1); ++q) acc2[q] = 0.f;
    auto store_tile = [&](int64_t tile) {
        const int64_t m0 = (tile * kWgThreads + tid) * COORDS;
        store_coords<COORDS>(a.ghat + m0, acc, m0, a.d);
        if constexpr (TWO) store_coords<COORDS>(a.ghat2 + m0, acc2, m0, a.d);
    };
    int64_t tile = blockIdx.x;
    if (a.n_chunks == 0) {  // nobody arrived
        for (; tile < a.n_tiles; tile += gridDim.x) store_tile(tile);
        return;
    }
    if constexpr (SCALES == 1) {
        for (int i = tid; i < a.n_arrived; i += kWgThreads) lds.worker[i] = (uint8_t)workers[i].worker;
        __syncthreads();
    }
    u32x4_t r[kDecPerThread];
    float aux[2] = {0.f, 0.f}, aux2[2] = {0.f, 0.f};
    auto request = [&](int64_t t, int c) {
        if (SCALES != 0) {  // weights or scales of the chunk's workers in the tile's buckets (= blocks)
            const int s0 = load_uniform(chunk_first + c), s1 = load_uniform(chunk_first + c + 1);
            const int64_t last_block = (a.d - 1) / kBlockCoords;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int e = tid + j * kWgThreads;
                const int slot = s0 + e / COORDS < s1 ? s0 + e / COORDS : s1 - 1;
                int64_t block = t * COORDS + e % COORDS;
                block = block < last_block ? block : last_block;
                if (SCALES == 1) {
                    aux[j] = a.scales[(int64_t)lds.worker[SCALES == 1 ? slot : 0] * a.nb + block];
                } else {
                    const int64_t row = (int64_t)a.block_layer[block] * a.n_arrived;
                    aux[j] = a.coef_layer[row + slot];
                    if (TWO) aux2[j] = a.coef2_layer[row + slot];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kDecPerThread; ++j) {
            const int p = tid + j * kWgThreads;
            const DecUnit un = units[c * kChunkUnits + p / kUnitPieces];
            // pieces past the end of the stream (coordinates past the end of the vector): its last one instead
            uint32_t at = (uint32_t)t * un.tile_pieces + (uint32_t)(p % kUnitPieces);
            at = at < un.pieces ? at : un.pieces - 1u;
            r[j] = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4_t*)un.codes + at);
        }
    };
    auto deliver = [&](int x) {
#pragma unroll
        for (int j = 0; j < kDecPerThread; ++j) lds_chunk[x][tid + j * kWgThreads] = r[j];
        if (SCALES != 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                lds_aux[SCALES ? x : 0][SCALES ? tid + j * kWgThreads : 0] = aux[j];
                if (SCALES == 2 && TWO)
                    lds_aux2[SCALES == 2 && TWO ? x : 0][SCALES == 2 && TWO ? tid + j * kWgThreads : 0] = aux2[j];
            }
        }
    };
    request(tile, 0);
    deliver(0);
    __syncthreads();
    int c = 0, x = 0;
    for (;;) {
        const bool tile_ends = c + 1 == a.n_chunks;
        const int c_next = tile_ends ? 0 : c + 1;
        const int64_t tile_next = tile_ends ? tile + gridDim.x : tile;
        const bool more = tile_next < a.n_tiles;
        if (more) request(tile_next, c_next);
        const int s0 = load_uniform(chunk_first + c), s1 = load_uniform(chunk_first + c + 1);
        auto record = [&](int slot) {  // coef, coef2, width, pos
            return *(const __attribute__((address_space(4))) u32x4_t*)(workers + slot);
        };
        u32x4_t next = record(s0);
        for (int slot = s0; slot < s1; ++slot) {
            const u32x4_t wk = next;
            next = record(slot + 1 < s1 ? slot + 1 : slot);  // in flight during this worker
            float c1 = __uint_as_float(wk.x), c2 = TWO ? __uint_as_float(wk.y) : 0.f;
            if (SCALES != 0) {
                const int e = (slot - s0) * COORDS + tid * COORDS / kWgThreads;
                const float s = lds_aux[x][e];
                if (SCALES == 1) {
                    c1 = c1 * s;
                    c2 = c2 * s;
                } else {
                    c1 = s;
                    if (TWO) c2 = lds_aux2[SCALES == 2 && TWO ? x : 0][SCALES == 2 && TWO ? e : 0];
                }
            }
            const uint32_t* part = reinterpret_cast<const uint32_t*>(&lds_chunk[x][wk.w * kUnitPieces]);
            uint32_t mask = wk.z;
            if (SCALES != 0) {  // the weights differ from lane to lane: one choice for the wave
                const bool halves1 = halves_exactly(c1), halves2 = !TWO || halves_exactly(c2);
                const uint64_t no = __builtin_amdgcn_ballot_w64(!(halves1 & halves2));
                mask = mask == 4u && no == 0 ? 1u : mask;
            }
            if (mask & 0x1Fu) decode_any<0, 4, COORDS, TWO>(mask, part, c1, c2, acc, acc2);
            if (mask & ~0x1Fu) {
                if (mask & 0x1E0u) decode_any<5, 8, COORDS, TWO>(mask, part, c1, c2, acc, acc2);
                if (mask & 0x1E00u) decode_any<9, 12, COORDS, TWO>(mask, part, c1, c2, acc, acc2);
                if (mask & 0x1E000u) decode_any<13, 16, COORDS, TWO>(mask, part, c1, c2, acc, acc2);
            }
        }
        if (tile_ends) {
            store_tile(tile);
#pragma unroll
            for (int q = 0; q < COORDS; ++q) acc[q] = 0.f;
#pragma unroll
            for (int q = 0; q < (TWO ? COORDS : 1); ++q) acc2[q] = 0.f;
        }
        if (!more) break;  // the same for every wave of the workgroup
        // the other buffer was last read before the barrier that ended the previous turn
        x ^= 1;
        deliver(x);
        __syncthreads();
        c = c_next;
        tile = tile_next;
    }
}

// The decode of a few workers: a lane owns 32 coordinates, which are `bits` whole words of a stream, and loads
// them right before they are used.  One request per wave is in flight, which bounds many workers (see above); for
// few of them the estimate's stores are most of the traffic, and here a lane writes a whole line of it.
template <int LO, int HI>
__device__ __forceinline__ void decode_direct(uint32_t mask, const global_u32* src, float c1, float (&acc)[32])
{
    if (mask & (1u << LO)) {
        constexpr int B = LO == 0 ? 2 : LO;
        uint32_t w[B];
        float none[1];
#pragma unroll
        for (int t = 0; t < B; ++t) w[t] = __builtin_nontemporal_load(src + t);
        if constexpr (LO == 0) decode_words_2bit<32, B, false>(w, 0.5f * c1, 0.f, acc, none);
        else decode_words<B, 32, B, false>(w, c1, 0.f, acc, none);
    }
    if constexpr (LO < HI) decode_direct<LO + 1, HI>(mask, src, c1, acc);
}

template <int SCALES>
__global__ __launch_bounds__(kWgThreads)
__attribute__((amdgpu_waves_per_eu(6, 6)))
void k_decode_direct(const DecWorker* __restrict__ workers, DecodeArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * kWgThreads + threadIdx.x;
    const int64_t m0 = t * 32, block = t >> 3;
    if (m0 >= a.d) return;
    float acc[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) acc[q] = 0.f;
    const float* layer_row = SCALES == 2 ? a.coef_layer + (int64_t)a.block_layer[block] * a.n_arrived : nullptr;
    for (int e = 0; e < a.n_arrived; ++e) {
        const DecWorker wk = load_uniform(workers + e);
        float c1 = wk.coef;
        uint32_t mask = wk.width;
        if (SCALES == 1) c1 = c1 * a.scales[(int64_t)wk.worker * a.nb + block];
        if (SCALES == 2) c1 = layer_row[e];
        if (SCALES != 0 && mask == 4u && __builtin_amdgcn_ballot_w64(!halves_exactly(c1)) == 0) mask = 1u;
        const global_u32* src = (const global_u32*)wk.codes + t * wk.bits;
        if (mask & 0x1Fu) decode_direct<0, 4>(mask, src, c1, acc);
        if (mask & 0x1E0u) decode_direct<5, 8>(mask, src, c1, acc);
        if (mask & 0x1FE00u) decode_direct<9, 16>(mask, src, c1, acc);
    }
    store_coords<32>(a.ghat + m0, acc, m0, a.d);
}

// ---- host side
template <bool TWO, int SCALES, int COORDS>
static void launch_decode_main(hipStream_t stream, const DecodeTables& tab, DecodeArgs a)
{
    a.n_tiles = (a.d + kWgThreads * COORDS - 1) / (kWgThreads * COORDS);
    const unsigned grid = (unsigned)decode_groups(a.n_tiles, a.n_chunks, decode_per_cu(sizeof(DecodeLds<TWO, SCALES>)));
    hipLaunchKernelGGL((k_decode<TWO, SCALES, COORDS>), dim3(grid), dim3(kWgThreads), 0, stream, tab.workers, tab.units,
                       tab.chunk_first, a);
}

template <bool TWO, int SCALES, int CAP>
static hipError_t launch_decode_cap(const DecodeStreams& in, int coords, const DecodeTables& tab, int n_layers,
                                    const float* scales, const Workspace* ws, DecodeArgs a, hipStream_t stream)
{
    DecodeList<CAP> list;
    list.n_arrived = in.n_arrived;
    list.groups = (uint32_t)((a.d + 127) / 128);
    const bool direct = !TWO && decode_is_direct(in.n_arrived, a.d);
    list.units_per_chunk = direct ? 0 : kDecChunkBytes / (32 * coords);
    list.unit_pieces = 2 * coords;
    int chunk = -1, fill = list.units_per_chunk;
    for (int i = 0; i < in.n_arrived; ++i) {  // consecutive workers, whole, as long as the chunk holds them
        const int b = in.bits[i];
        if (fill + b > list.units_per_chunk) {
            ++chunk;
            fill = 0;
        }
        list.codes[i] = in.codes[i];
        list.w[i] = in.w[i];
        list.v[i] = in.v[i];
        list.bits[i] = in.bits[i];
        list.worker[i] = in.worker[i];
        list.chunk[i] = (uint8_t)chunk;
        list.pos[i] = (uint8_t)fill;
        fill += b;
    }
    a.n_arrived = in.n_arrived;
    a.n_chunks = chunk + 1;
    if (in.n_arrived > 0) {
        hipLaunchKernelGGL((k_decode_table<CAP, SCALES, TWO>), dim3(SCALES == 2 ? n_layers : 1), dim3(kWgThreads), 0,
                           stream, list, scales, n_layers, tab, SCALES == 2 ? ws->coef_layer : nullptr,
                           SCALES == 2 ? ws->coef2_layer : nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if constexpr (!TWO) {
        if (direct) {
            const int64_t lanes = (a.d + 31) / 32;
            hipLaunchKernelGGL((k_decode_direct<SCALES>), dim3((unsigned)((lanes + kWgThreads - 1) / kWgThreads)),
                               dim3(kWgThreads), 0, stream, tab.workers, a);
            return hipGetLastError();
        }
        if (coords == 16) launch_decode_main<TWO, SCALES, 16>(stream, tab, a);
    }
    if (coords == 8) launch_decode_main<TWO, SCALES, 8>(stream, tab, a);
    return hipGetLastError();
}

template <bool TWO, int SCALES>
static hipError_t launch_decode_scales(const DecodeStreams& in, const DecodeTables& tab, int n_layers,
                                       const float* scales, const Workspace* ws, const DecodeArgs& a, hipStream_t stream)
{
    int sum_bits = 0;
    for (int i = 0; i < in.n_arrived; ++i) sum_bits += in.bits[i];
    const int coords = decode_coords(a.d, TWO, SCALES != 0, sum_bits);
    // the launch copies its arguments at about 1.7 ns a byte: 20 bytes per worker it has room for
    if (in.n_arrived <= 16) return launch_decode_cap<TWO, SCALES, 16>(in, coords, tab, n_layers, scales, ws, a, stream);
    if (in.n_arrived <= 64) return launch_decode_cap<TWO, SCALES, 64>(in, coords, tab, n_layers, scales, ws, a, stream);
    return launch_decode_cap<TWO, SCALES, kArgWorkers>(in, coords, tab, n_layers, scales, ws, a, stream);
}

// tables inside a block of decode_table_bytes(n) bytes
static DecodeTables decode_tables(void* base, int n)
{
    char* p = static_cast<char*>(base);
    DecodeTables t;
    t.workers = reinterpret_cast<DecWorker*>(p);
    t.units = reinterpret_cast<DecUnit*>(p + sizeof(DecWorker) * (size_t)n);
    t.chunk_first = reinterpret_cast<int*>(p + sizeof(DecWorker) * (size_t)n + sizeof(DecUnit) * (size_t)decode_units(n));
    return t;
}

hipError_t launch_decode(int n, int64_t d, const DecodeStreams& in, bool two, const float* scales, int64_t nb,
                         const Workspace& ws, float* ghat, float* ghat2, hipStream_t stream)
{
    DecodeArgs a{};
    a.d = d;
    a.ghat = ghat;
    a.ghat2 = ghat2;
    a.scales = scales;
    a.nb = nb;
    a.block_layer = ws.block_layer;
    a.coef_layer = ws.coef_layer;
    a.coef2_layer = ws.coef2_layer;
    const DecodeTables tab = decode_tables(ws.dec, n);
    if (ws.n_layers > 0)
        return two ? launch_decode_scales<true, 2>(in, tab, ws.n_layers, scales, &ws, a, stream)
                   : launch_decode_scales<false, 2>(in, tab, ws.n_layers, scales, &ws, a, stream);
    if (nb > 0)
        return two ? launch_decode_scales<true, 1>(in, tab, 0, scales, &ws, a, stream)
                   : launch_decode_scales<false, 1>(in, tab, 0, scales, &ws, a, stream);
    return two ? launch_decode_scales<true, 0>(in, tab, 0, scales, &ws, a, stream)
               : launch_decode_scales<false, 0>(in, tab, 0, scales, &ws, a, stream);
}

// ---------------------------------------------------------------------------------------
// Decode for callers that cannot allocate (HIP graph capture, tight serving loops): the tables of
// arrived workers, which agc_decode keeps in the context's workspace, live in a fixed device array
// instead.  Each GPU holds its own copy of the array at its own address; host code only ever uses
// the address that hipGetSymbolAddress returned for the device that was current.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[decode_table_bytes(kMaxWorkers)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices];  // per device: the device address of `scratch`, null = not resolved yet
}  // namespace

hipError_t launch_decode_static(int64_t d, const DecodeStreams& in, const float* scales, int64_t nb, float* ghat,
                                hipStream_t stream)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* base = nullptr;
    {
        std::lock_guard<std::mutex> hold(g_scratch_lock);
        if (!g_scratch_ptr[dev]) {  // first call on this device, which is the current one
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!p) return hipErrorInvalidSymbol;
            g_scratch_ptr[dev] = p;
        }
        base = g_scratch_ptr[dev];
    }
    // the prologue rewrites every entry that the decode kernel reads, so nothing of the previous
    // call's contents has to be cleared
    DecodeArgs a{};
    a.d = d;
    a.ghat = ghat;
    a.scales = scales;
    a.nb = nb;
    const DecodeTables tab = decode_tables(base, kMaxWorkers);
    return nb > 0 ? launch_decode_scales<false, 1>(in, tab, 0, scales, nullptr, a, stream)
                  : launch_decode_scales<false, 0>(in, tab, 0, scales, nullptr, a, stream);
}

// Adam with the two-track estimates (Sec. V): first moment from the unbiased estimate, second
// moment from the square of the variance-reduced one.  corr1 = 1 - beta1^t, corr2 = 1 - beta2^t.
__global__ __launch_bounds__(kWgThreads) void k_adam_update(float* beta, float* m1, float* m2,
                                                            const float* __restrict__ ghat,
                                                            const float* __restrict__ ghat2, float lr, float beta1,
                                                            float beta2, float eps, float corr1, float corr2,
                                                            int64_t d)
{
    const int64_t i = (int64_t)blockIdx.x * kWgThreads + threadIdx.x;
    if (i >= d) return;
    const float g = ghat[i], h = ghat2[i];
    const float a = fmaf(beta1, m1[i], (1.0f - beta1) * g);
    const float b = fmaf(beta2, m2[i], (1.0f - beta2) * (h * h));
    m1[i] = a;
    m2[i] = b;
    beta[i] = beta[i] - lr * (a / corr1) / (sqrtf(b / corr2) + eps);
}

hipError_t launch_adam_update(float* beta, float* m1, float* m2, const float* ghat, const float* ghat2,
                              float lr, float beta1, float beta2, float eps, float corr1, float corr2,
                              int64_t d, hipStream_t stream)
{
    hipLaunchKernelGGL(k_adam_update, dim3((unsigned)((d + kWgThreads - 1) / kWgThreads)), dim3(kWgThreads), 0,
                       stream, beta, m1, m2, ghat, ghat2, lr, beta1, beta2, eps, corr1, corr2, d);
    return hipGetLastError();
}

}  // namespace agc
