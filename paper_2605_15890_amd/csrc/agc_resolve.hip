// k_resolve: codes and estimate of the signs and records that k_sketch has left (agc_sketch.h), once the scales are known.
#include "agc_device.h"
#include "agc_kernels.h"
#include "agc_quantize.h"

namespace agc {

struct ResolveArgs {
    int n;
    int64_t d;
    uint32_t key0, key1, step_lo, step_hi;
    float* ghat;
    int stage_bits;
    SketchDev sk;
};

constexpr int kClaims = 128;  // claim words of a wave; a coordinate's is its low seven bits

// Sign bits of 32 codes -> the words of the stream that hold them, at the top bits of the codes.  Word w of 32 codes of B
// bits (of sixteen, where B is even: half a wave each) holds the signs from code 32 w / B on; they are spread
// by doubling the gaps.
template <int B, int COUNT, int STEP>
__device__ __forceinline__ uint32_t spread_bits(uint32_t x)  // bit c -> bit c * B for c < COUNT
{
    if constexpr (STEP > 0) {
        if constexpr (STEP < COUNT) {
            constexpr uint64_t group = (1ull << STEP) - 1;
            uint64_t mask = 0;
#pragma unroll
            for (int c = 0; c * STEP < COUNT; ++c) mask |= group << (c * STEP * B);
            x = (x | (x << (STEP * (B - 1)))) & (uint32_t)mask;
        }
        x = spread_bits<B, COUNT, STEP / 2>(x);
    }
    return x;
}
template <int B, int W>
__device__ __forceinline__ uint32_t sign_word(uint32_t signs)
{
    constexpr int first = 32 * W / B, at = first * B + B - 1 - 32 * W, count = (31 - at) / B + 1;
    const uint32_t x = (signs >> first) & (count >= 32 ? ~0u : (1u << count) - 1u);
    return spread_bits<B, count, 16>(x) << at;
}
template <int B, int... Ws>
__device__ __forceinline__ void or_sign_words(uint32_t* dst, uint32_t signs, std::integer_sequence<int, Ws...>)
{
    ((dst[Ws] |= sign_word<B, Ws>(signs)), ...);
}
// the signs of one worker for the workgroup's 1024 coordinates; part: the worker's words in the staging area
template <int B>
__device__ __forceinline__ void or_signs(uint32_t* part, uint32_t signs, int lane)
{
    if constexpr (B % 2 == 0) {
        or_sign_words<B>(part + (lane & 31) * B + (lane >> 5) * (B / 2), signs >> (16 * (lane >> 5)),
                         std::make_integer_sequence<int, B / 2>{});
    } else if (lane < 32) {
        or_sign_words<B>(part + lane * B, signs, std::make_integer_sequence<int, B>{});
    }
}
template <int LO, int HI>
__device__ __forceinline__ void or_signs_any(int b, uint32_t* part, uint32_t signs, int lane)  // b is wave-uniform
{
    if constexpr (LO == HI) {
        or_signs<LO>(part, signs, lane);
    } else {
        constexpr int mid = LO == 2 && HI > 4 ? (HI > 8 ? 8 : 4) : (LO + HI) / 2;
        if (b <= mid) or_signs_any<LO, mid>(b, part, signs, lane);
        else or_signs_any<mid + 1, HI>(b, part, signs, lane);
    }
}

// What bounds it: 0.95 GB in and out at 64 workers x 25.6 M (205 MB of signs, 30 of records, 614 of codes, 102 of estimate) in
// 0.31 ms, 3 TB/s; latency is most of the rest: waves wait 0.47 of their time, vector ALU 0.35 busy (counters of the interval
// code).  Signs lane by lane, with an LDS atomic for every
// word that two lanes share, took 0.80 ms; whole words per lane 0.41; with the fill's end looked up in LDS instead of worker
// by worker in memory 0.31.
//
// A group of four blocks per workgroup.  A wave first ORs the levels of its block's records into the staging area of
// k_quantize, one record per lane; then the waves share the workers, add their signs and write them out.  The estimate is
// summed in LDS, where only levels above zero change it (the running sums start at +0, and finite weights times a zero
// level leave them as they are).  Records are ordered by worker and a worker has a coordinate once, so the sums take
// their terms in ascending order of workers if, of the lanes that hold the same coordinate, the lowest goes
// first: lanes claim the coordinate with their number by an atomic minimum, in rounds.
template <bool FUSE>
__global__ __launch_bounds__(kWgThreads) void k_resolve(const WorkerQ* __restrict__ wq, ResolveArgs a)
{
    // stage_pieces(a.stage_bits, 4) pieces, then [n] records of 16 bytes, then (FUSE) [4][256] sums and [4][kClaims] claims, then
    // [4][8 * n + 8] signs
    extern __shared__ __attribute__((aligned(16))) uint32_t lds_stage[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t wg = blockIdx.x;
    const int64_t block = wg * kQuantWaves + wave;
    const int64_t base = block * (int64_t)kBlockCoords;
    const bool has_block = base < a.d;
    struct Counts { int c[4]; };
    const Counts counts = load_uniform(reinterpret_cast<const Counts*>(a.sk.counts + 4 * wg));
    if (load_uniform(a.sk.state) != 0u) return;  // all are left to k_quantize
    if ((counts.c[0] | counts.c[1] | counts.c[2] | counts.c[3]) < 0) {
        if (threadIdx.x == 0)
            a.sk.left[__hip_atomic_fetch_add(a.sk.state + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = (uint32_t)wg;
        return;
    }
    const int np = stage_pieces(a.stage_bits, kQuantWaves);
    u32x4_t* pieces = reinterpret_cast<u32x4_t*>(lds_stage);
    for (int p = threadIdx.x; p < np; p += kQuantThreads) pieces[p] = u32x4_t{0u, 0u, 0u, 0u};
    u32x4_t* table = pieces + np;  // multiplier, weight, bits with arrived and flush, first word of the worker in the area
    for (int i = threadIdx.x; i < a.n; i += kQuantThreads) {
        const WorkerQ q = wq[i];
        table[i] = u32x4_t{__float_as_uint(q.inv16), __float_as_uint(q.coef), q.bits | (q.arrived << 8) | (q.flush << 9), 4u * q.stage_piece};
    }
    float* sums = reinterpret_cast<float*>(table + a.n) + wave * kBlockCoords;
    uint32_t* claims = reinterpret_cast<uint32_t*>(table + a.n) + kQuantWaves * kBlockCoords + wave * kClaims;
    if (FUSE) {
        *reinterpret_cast<u32x4_t*>(sums + 4 * lane) = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < kClaims; t += kWave) claims[t + lane] = 0xFFFFFFFFu;
    }
    const int sign_stride = 8 * a.n + 8;  // dwords of a block; the eight keep the four blocks in different banks
    uint32_t* signs = lds_stage + 4 * np + 4 * a.n + (FUSE ? kQuantWaves * (kBlockCoords + kClaims) : 0);
    if (has_block) {
        const u32x4_t* planes = reinterpret_cast<const u32x4_t*>(a.sk.planes) + block * (int64_t)(a.sk.chunks * kWave);
        u32x4_t* to = reinterpret_cast<u32x4_t*>(signs + wave * sign_stride);
        for (int p = lane; p < 2 * a.n; p += kWave) to[p] = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4_t*)planes + p);
    } else {
        for (int p = lane; p < 8 * a.n; p += kWave) signs[wave * sign_stride + p] = 0u;
    }
    __syncthreads();
    const int64_t groups_left = (a.d + 127) / 128 - 2 * kQuantWaves * wg;
    const int wg_groups = groups_left >= 2 * kQuantWaves ? 2 * kQuantWaves : (int)groups_left;
    const uint32_t ctr_base = (uint32_t)(base >> 2);
    const int count = wave == 0 ? counts.c[0] : wave == 1 ? counts.c[1] : wave == 2 ? counts.c[2] : counts.c[3];
    const uint2* recs = a.sk.recs + block * (int64_t)a.sk.cap;
    int ptr = 0;
    auto record = [&](int from) {
        const int p = from + lane;
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        const u32x2_t v = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x2_t*)(recs + (p < count ? p : 0)));
        return make_uint2(v.x, v.y);
    };
    uint2 rec = make_uint2(0u, 0u);
    if (count > 0) rec = record(0);
    int i = 0;
    while (i < a.n) {  // one turn per fill of the staging area
        const int first = i;
        for (;; i += kWave) {  // up to the worker that ends the fill; the last of all has the flag
            const bool ends = i + lane < a.n && (table[i + lane < a.n ? i + lane : i].z & 512u) != 0u;
            const uint64_t m = __builtin_amdgcn_ballot_w64(ends);
            if (m == 0) continue;
            i += __builtin_ctzll(m) + 1;
            break;
        }
        // records of the fill's workers
        while (ptr < count) {
            const uint2 ahead = record(ptr + kWave < count ? ptr + kWave : ptr);
            const uint32_t worker = (rec.y >> 8) & 255u;
            const bool mine = lane < count - ptr && (int)worker < i;
            const uint64_t m = __builtin_amdgcn_ballot_w64(mine);
            if (m == 0) break;
            const u32x4_t t = table[worker];
            const uint32_t b = t.z & 255u, coord = rec.y & 255u;
            const uint32_t L = (1u << (b - 1u)) - 1u;
            const float f = __uint_as_float(rec.x);
            const float T = grid_pos<false>(f, __uint_as_float(t.x));
            bool tie;
            uint32_t level = round_primary(T, rec.y >> 16, L, tie);
            if (__any(tie && mine)) {
                uint32_t r2[4];
                philox4x32_10(ctr_base + (coord >> 2), 0x80000000u | worker, a.step_lo, a.step_hi, a.key0, a.key1, r2);
                const uint32_t r = (coord & 2u) ? ((coord & 1u) ? r2[3] : r2[2]) : ((coord & 1u) ? r2[1] : r2[0]);
                if (tie) level = round_tied(T, r, L);
            }
            bool add = mine && level != 0u;
            if (add) {
                const uint32_t bitpos = coord * b;
                uint32_t* at = lds_stage + t.w + (uint32_t)wave * 8u * b + (bitpos >> 5);
                const uint64_t v = (uint64_t)level << (bitpos & 31u);
                atomicOr(at, (uint32_t)v);
                if ((uint32_t)(v >> 32) != 0u) atomicOr(at + 1, (uint32_t)(v >> 32));
            }
            if constexpr (FUSE) {
                add = add && (t.z & 256u) != 0u;
                const float v = __uint_as_float(__float_as_uint((float)level) | (rec.x & 0x80000000u));
                const float coef = __uint_as_float(t.y);
                uint32_t* claim = claims + (coord & (kClaims - 1));
                while (__any(add)) {  // the lowest lane that is left always succeeds
                    if (add) atomicMin(claim, (uint32_t)lane);
                    asm volatile("" ::: "memory");  // lanes read what others have written; LDS serves a wave in order
                    const bool go = add && *claim == (uint32_t)lane;
                    if (go) {
                        sums[coord] = fmaf(coef, v, sums[coord]);
                        *claim = 0xFFFFFFFFu;
                    }
                    asm volatile("" ::: "memory");
                    add = add && !go;
                }
            }
            const int taken = __builtin_popcountll(m);
            ptr += taken;
            rec = taken == kWave ? ahead : record(ptr);
        }
        __syncthreads();
        const uint32_t* my_signs = signs + ((lane & 31) >> 3) * sign_stride + (lane & 7);
        const int j0 = first + wave < a.n ? first + wave : a.n - 1;
        u32x4_t t_next = table[j0];
        uint32_t s_next = my_signs[8 * j0];
        for (int j = first + wave; j < i; j += kQuantWaves) {  // as store_fill shares them
            const uint32_t b = __builtin_amdgcn_readfirstlane(t_next.z & 255u);
            uint32_t* part = lds_stage + __builtin_amdgcn_readfirstlane(t_next.w);
            const uint32_t s = s_next;
            const int ahead = j + kQuantWaves < a.n ? j + kQuantWaves : a.n - 1;
            t_next = table[ahead];
            s_next = my_signs[8 * ahead];
            or_signs_any<2, 16>((int)b, part, s, lane);
        }
        asm volatile("" ::: "memory");  // lanes read what others have written
        store_fill<kQuantWaves, true>(lds_stage, wq, first, i - 1, wave, lane, wg, wg_groups);
        if (i < a.n) __syncthreads();  // the area is reused by the next fill
    }
    if constexpr (FUSE) {
        if (has_block) {
            const int64_t left = a.d - base - 4 * lane;
            const u32x4_t s = *reinterpret_cast<const u32x4_t*>(sums + 4 * lane);
            float* dst = a.ghat + base + 4 * lane;
            if (left >= 4) *reinterpret_cast<u32x4_t*>(dst) = s;
            else
                for (int t = 0; t < left; ++t) dst[t] = sums[4 * lane + t];
        }
    }
}

hipError_t launch_resolve(int n, int64_t d, const Workspace& ws, const SketchDev& sk, const QuantStreams& out, uint64_t seed,
                          uint64_t step, float* ghat, hipStream_t stream)
{
    const ResolveArgs a{n, d, (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32), ghat,
                        out.stage_bits, sk};
    if (out.stage_bits < 1 || out.stage_bits > kStageBits) return hipErrorInvalidValue;
    const dim3 g((unsigned)((d + 1023) / 1024)), b(kQuantThreads);
    const unsigned lds = 16u * (unsigned)(stage_pieces(out.stage_bits, kQuantWaves) + n) +
                         (ghat ? 4u * (unsigned)(kQuantWaves * (kBlockCoords + kClaims)) : 0u) +
                         4u * (unsigned)(kQuantWaves * (8 * n + 8));
    if (ghat) hipLaunchKernelGGL((k_resolve<true>), g, b, lds, stream, ws.wq, a);
    else hipLaunchKernelGGL((k_resolve<false>), g, b, lds, stream, ws.wq, a);
    return hipGetLastError();
}

}  // namespace agc
