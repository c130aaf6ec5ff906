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
// 984, quantize pass 1420), 1565 with one: sample and bounds 11 + 5, k_sketch 1210-1240, groups and finalize 13,
// k_resolve 310, the quantize pass that finds nothing left 7.  A step whose bounds do not hold pays for both forms (some 2670).
// Values that are not alike everywhere, two reads | one: rows of 16384 with the first 256 values 20 times the others, six bits,
// 64 x 25.6 M 2500 | 1950, 50 x 5.4 M 480 | 437, 64 x 5.4 M three bits 541 | 402; sixty layers of magnitudes up to 1000 apart,
// eight bits, 64 x 25.6 M 2552 | 2108.  What stays slower: at 64 x 1 M the second pass takes 27 us for however few blocks, so a
// norm in a 64th of the vector or less, 132 | 139, and such rows, 132 | 141, lose what alike values gain, 132 | 108.
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
    double* part_sq;       // [segment][worker]
    SketchDev sk;
};

// The norm's exchange-add over the 64 lanes (wave_butterfly_add) for four workers at once: after the first exchange a
// lane goes on with one of two workers only, after the second with one of four, so that the later ones are shared.  Every
// worker's sums are the same pairs as alone.
__device__ __forceinline__ double sum_rows_of_four(double v)  // lane l: worker l & 3, sum of its quad -> of the wave
{
    return exchange_halves(exchange_quads(v));
}

struct EpiSketch {
    static constexpr bool kStoresPerWorker = false;
    static constexpr bool kWantsZeros = true;
    static constexpr int kPrefetchRows = AGC_PREFETCH_ROWS;
    const float* lo_mult;  // [n], scalar reads
    uint32_t key0, key1, step_lo, step_hi;
    double* acc;           // this wave's LDS slices: [n]
    uint32_t* plane;       // [worker][8]: 256 signs in the order of the coordinates
    uint2* recs;           // [cap]
    int cap, n;
    int lane;
    uint32_t ctr0;
    int count;             // wave-uniform: records so far, with those that did not fit
    uint32_t keep2, keep3; // second half of the pair's Philox block
    uint32_t word;         // the lane's signs of the last eight workers, coordinate q of the newest at bit q
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
    uint32_t keep0, keep1;
    __device__ __forceinline__ void draw(int i)
    {
        uint32_t o[4];
        philox4x32_10(ctr0, (uint32_t)i >> 1, step_lo, step_hi, key0, key1, o);
        keep0 = o[0];
        keep1 = o[1];
        keep2 = o[2];
        keep3 = o[3];
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
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.w), 31);
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.z), 31);
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.y), 31);
        word = __builtin_amdgcn_alignbit(word, __float_as_uint(f.x), 31);
        if ((i & 7) == 7 || i == n - 1) store_signs(i);
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

// What bounds it: stores among reads.  With the cyclic code the bare row walk takes 0.96 ms, the kernel without its stores
// 1.04, with the 205 MB of signs 1.21 (plain stores 1.235, non-temporal 1.218, written through as well 1.21); without
// the Philox rounds or the sums of squares it is not faster.  Three, four, five, six waves per SIMD: 1.47, 1.24, 1.215,
// 1.32 ms; four leave the most room for records.  Four workers' sums share their exchanges because vector
// instructions still count at that occupancy: 76 per worker and wave (the sums of each worker alone: 90).
//
// One wave per block of 256 coordinates, four blocks of a segment of the norm's tree per workgroup.
// LDS: [4][n] doubles, [4][4 * chunks][64] dwords of signs, [4][cap] records.
template <int S>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(S == 0 ? 1 : 4, S == 0 ? 8 : 4))) void k_sketch(
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
        EpiSketch epi{lo_mult, a.key0, a.key1, a.step_lo, a.step_hi, acc, plane, recs, a.sk.cap, a.n, lane,
                      (uint32_t)((base + 4 * lane) >> 2), 0, 0u, 0u, 0u, 0.0, 0.0, load_uniform(lo_mult), 0u, 0u};
        encode_block<S>(G + base, a.ldg, a.n, a.k, CsrView{row_ptr, col, val, a.win}, lc, epi);
        epi.finish();
        // what this wave's lanes have left in LDS leaves in long runs, by the store policy of the payload
        asm volatile("" ::: "memory");  // the lanes read what others have written
        const u32x4_t* signs = reinterpret_cast<const u32x4_t*>(plane);
        const __amdgpu_buffer_rsrc_t out = uniform_buffer(a.sk.planes + block * (int64_t)(4 * a.sk.chunks * kWave), 32 * a.n);
        for (int p = lane; p < 2 * a.n; p += kWave)
            __builtin_amdgcn_raw_buffer_store_b128(signs[p], out, 16 * p, 0, kPayloadStorePolicy);
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

template <int S>
static hipError_t launch_sketch_s(const float* G, const CodeDev& code, const SketchArgs& a, hipStream_t stream)
{
    hipLaunchKernelGGL((k_sketch<S>), dim3((unsigned)((a.d + 1023) / 1024)), dim3(kWgThreads), sketch_lds_bytes(a.n, a.sk.cap),
                       stream, G, code.row_ptr, code.col, code.val, a.sk.lo_mult, a);
    return hipGetLastError();
}

}  // namespace agc
