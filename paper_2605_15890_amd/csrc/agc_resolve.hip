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

constexpr int kClaims = kBlockCoords;  // claim words of a wave, one for every coordinate of its block

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
template <int B, int N, int... Ws>
__device__ __forceinline__ void sign_words(uint32_t (&v)[N], uint32_t signs, std::integer_sequence<int, Ws...>)
{
    ((v[Ws] |= sign_word<B, Ws>(signs)), ...);
}
// One worker's codes of the workgroup's 1024 coordinates: levels from the staging area, signs ORed in, stored to its stream.
// signs: 32 codes' worth, those of run lane mod 32.  Widths that are even: sixteen codes are whole words, which a lane takes from
// the area, completes and stores, half a wave the first sixteen of every run and the other half the second, so that the wave
// stores one run of bytes.  Odd ones: half the wave completes 32 codes each in the area, and the wave stores 16-byte pieces.
// Runs past the end of the stream lie past `bytes` and are dropped by the range check, which never parts what a lane stores.
template <int B>
__device__ __forceinline__ void store_worker(uint32_t* part, uint32_t signs, int lane, bool clear, __amdgpu_buffer_rsrc_t out)
{
    if constexpr (B % 2 == 0) {
        constexpr int W = B / 2;
        uint32_t* at = part + (lane & 31) * B + (lane >> 5) * W;
        uint32_t v[W];
#pragma unroll
        for (int t = 0; t < W; ++t) v[t] = at[t];
        sign_words<B>(v, signs >> (16 * (lane >> 5)), std::make_integer_sequence<int, W>{});
        if (clear) {
#pragma unroll
            for (int t = 0; t < W; ++t) at[t] = 0u;
        }
        const int off = (lane & 31) * (4 * B) + (lane >> 5) * (2 * B);
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
        int t = 0;
        if constexpr (W >= 4) {
            __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{v[0], v[1], v[2], v[3]}, out, off, 0, kPayloadStorePolicy);
            t = 4;
        }
        if constexpr (W >= 4 ? W % 4 == 1 : W == 1) __builtin_amdgcn_raw_buffer_store_b32(v[W - 1], out, off + 4 * t, 0, kPayloadStorePolicy);
        if constexpr (W >= 4 ? W % 4 == 2 : W == 2) __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{v[W - 2], v[W - 1]}, out, off + 4 * t, 0, kPayloadStorePolicy);
        if constexpr (W >= 4 ? W % 4 == 3 : W == 3) __builtin_amdgcn_raw_buffer_store_b96(u32x3_t{v[W - 3], v[W - 2], v[W - 1]}, out, off + 4 * t, 0, kPayloadStorePolicy);
        if constexpr (W == 8) __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{v[4], v[5], v[6], v[7]}, out, off + 16, 0, kPayloadStorePolicy);
    } else {
        if (lane < 32) {
            uint32_t* at = part + lane * B;
            uint32_t v[B];
#pragma unroll
            for (int t = 0; t < B; ++t) v[t] = at[t];
            sign_words<B>(v, signs, std::make_integer_sequence<int, B>{});
#pragma unroll
            for (int t = 0; t < B; ++t) at[t] = v[t];
        }
        asm volatile("" ::: "memory");  // lanes read what others have written
        u32x4_t* pieces = reinterpret_cast<u32x4_t*>(part);
#pragma unroll
        for (int p0 = 0; p0 < 8 * B; p0 += kWave) {
            const int p = p0 + lane;
            if (p < 8 * B) {
                __builtin_amdgcn_raw_buffer_store_b128(pieces[p], out, 16 * p, 0, kPayloadStorePolicy);
                if (clear) pieces[p] = u32x4_t{0u, 0u, 0u, 0u};
            }
        }
        asm volatile("" ::: "memory");
    }
}
template <int LO, int HI>
__device__ __forceinline__ void store_worker_any(int b, uint32_t* part, uint32_t signs, int lane, bool clear, __amdgpu_buffer_rsrc_t out)
{  // b is wave-uniform
    if constexpr (LO == HI) {
        store_worker<LO>(part, signs, lane, clear, out);
    } else {
        constexpr int mid = LO == 2 && HI > 4 ? (HI > 8 ? 8 : 4) : (LO + HI) / 2;
        if (b <= mid) store_worker_any<LO, mid>(b, part, signs, lane, clear, out);
        else store_worker_any<mid + 1, HI>(b, part, signs, lane, clear, out);
    }
}

// What bounds it: latency; a workgroup is one chain of requests, LDS operations and barriers, and what counts is how many
// share a compute unit.  64 workers x 25.6 M, interval code, Euclidean: 0.95 GB in and out (205 MB of signs, 30 of records, 614 of
// codes, 102 of estimate) in 232 us, 4.1 TB/s;  largest magnitude with heavy tails, 450 records a block: 1.28 GB in 374.
// All workers' codes in one fill, four workgroups a compute unit, records one chunk ahead, every width completed in LDS and claims for
// two coordinates each: 317 and 450 us, 104 for 84 at 50 workers x 5.4 M without estimate.  Signs worker by worker from
// memory instead of LDS left room for eight workgroups and took 364 and 491.
//
// A group of four blocks per workgroup.  A wave first ORs the levels of its block's records into the staging area of
// k_quantize, one record per lane; then the waves share the workers, add their signs and store them.  The estimate is
// summed in LDS, where only levels above zero change it (the running sums start at +0, and finite weights times a zero
// level leave them as they are).  Records are ordered by worker and a worker has a coordinate once, so the sums take
// their terms in ascending order of workers if, of the lanes that hold the same coordinate, the lowest goes
// first: lanes claim the coordinate with their number by an atomic minimum, in rounds.
constexpr int kChunksAhead = 4;  // of 64 records
template <bool FUSE>
__global__ __launch_bounds__(kWgThreads) __attribute__((amdgpu_waves_per_eu(kResolveWgs, 8))) void k_resolve(const WorkerQ* __restrict__ wq, ResolveArgs a)
{
    // resolve_pieces(a.stage_bits) pieces, then [n] records of 16 bytes, then (FUSE) [4][256] sums and [4][kClaims] claims, then
    // [4][8 * n + 8] signs
    extern __shared__ __attribute__((aligned(16))) uint32_t lds_stage[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t wg = blockIdx.x;
    const int64_t block = wg * kQuantWaves + wave;
    const int64_t base = block * (int64_t)kBlockCoords;
    if (load_uniform(a.sk.state) != 0u) return;  // all are left to k_quantize
    struct Counts { int c[4]; };
    const Counts counts = load_uniform(reinterpret_cast<const Counts*>(a.sk.counts + 4 * wg));
    // what does not depend on the counts is requested before they are looked at: the first records, signs and the table
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(1))) u32x2_t* global_u32x2_t;
    const bool has_block = base < a.d;
    const global_u32x2_t recs = (global_u32x2_t)(a.sk.recs + (has_block ? block : 0) * (int64_t)a.sk.cap);
    auto record = [&](int from, int end) { return __builtin_nontemporal_load(recs + (from + lane < end ? from + lane : 0)); };
    u32x2_t rec[kChunksAhead];
#pragma unroll
    for (int t = 0; t < kChunksAhead; ++t) rec[t] = record(t * kWave, a.sk.cap);
    // the signs of the wave's block: [worker][8] words, two pieces of 16 bytes a worker
    const __attribute__((address_space(1))) u32x4_t* planes =
        (const __attribute__((address_space(1))) u32x4_t*)a.sk.planes + (has_block ? block : 0) * (int64_t)(a.sk.chunks * kWave);
    u32x4_t sign[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) sign[t] = __builtin_nontemporal_load(planes + (t * kWave + lane < 2 * a.n ? t * kWave + lane : 0));
    if ((counts.c[0] | counts.c[1] | counts.c[2] | counts.c[3]) < 0) {
        if (threadIdx.x == 0)
            a.sk.left[__hip_atomic_fetch_add(a.sk.state + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = (uint32_t)wg;
        return;
    }
    const int np = resolve_pieces(a.stage_bits);
    u32x4_t* pieces = reinterpret_cast<u32x4_t*>(lds_stage);
    u32x4_t* table = pieces + np;  // multiplier, weight, bits with arrived and end of a fill, first word of the worker in the area
    if ((int)threadIdx.x < a.n) table[threadIdx.x] = reinterpret_cast<const u32x4_t*>(a.sk.table)[threadIdx.x];  // n <= 256
    for (int p = threadIdx.x; p < np; p += kQuantThreads) pieces[p] = u32x4_t{0u, 0u, 0u, 0u};
    float* sums = reinterpret_cast<float*>(table + a.n) + wave * kBlockCoords;
    uint32_t* claims = reinterpret_cast<uint32_t*>(table + a.n) + kQuantWaves * kBlockCoords + wave * kClaims;
    if (FUSE) {
        *reinterpret_cast<u32x4_t*>(sums + 4 * lane) = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < kClaims; t += kWave) claims[t + lane] = 0xFFFFFFFFu;
    }
    const int sign_stride = 8 * a.n + 8;  // dwords of a block; the eight keep the four blocks in different banks
    uint32_t* signs = lds_stage + 4 * (np + a.n) + (FUSE ? kQuantWaves * (kBlockCoords + kClaims) : 0);
    {
        u32x4_t* to = reinterpret_cast<u32x4_t*>(signs + wave * sign_stride);
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (t * kWave + lane < 2 * a.n) to[t * kWave + lane] = has_block ? sign[t] : u32x4_t{0u, 0u, 0u, 0u};
        for (int p = 2 * kWave + lane; p < 2 * a.n; p += kWave) to[p] = has_block ? __builtin_nontemporal_load(planes + p) : u32x4_t{0u, 0u, 0u, 0u};
    }
    const uint32_t* my_signs = signs + ((lane & 31) >> 3) * sign_stride + (lane & 7);
    __syncthreads();
    const int64_t groups_left = (a.d + 127) / 128 - 2 * kQuantWaves * wg;
    const int wg_groups = groups_left >= 2 * kQuantWaves ? 2 * kQuantWaves : (int)groups_left;
    const uint32_t ctr_base = (uint32_t)(base >> 2);
    const int count = wave == 0 ? counts.c[0] : wave == 1 ? counts.c[1] : wave == 2 ? counts.c[2] : counts.c[3];
    int ptr = 0;  // first record of the chunk in rec[0]
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
            const uint32_t value = rec[0].x, what = rec[0].y;
            const uint32_t worker = (what >> 8) & 255u;
            const bool valid = lane < count - ptr, mine = valid && (int)worker < i && (int)worker >= first;
            if (__builtin_amdgcn_ballot_w64(mine) == 0) break;  // all of the chunk's are for later fills
            const u32x4_t t = table[mine ? worker : 0u];
            const uint32_t b = t.z & 255u, coord = what & 255u;
            const uint32_t L = (1u << (b - 1u)) - 1u;
            const float T = grid_pos<false>(__uint_as_float(value), __uint_as_float(t.x));
            bool tie;
            uint32_t level = round_primary(T, what >> 16, L, tie);
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
                const float v = __uint_as_float(__float_as_uint((float)level) | (value & 0x80000000u));
                const float coef = __uint_as_float(t.y);
                uint32_t* claim = claims + coord;
                while (__any(add)) {  // the lowest lane that is left always succeeds
                    if (add) atomicMin(claim, (uint32_t)lane);
                    asm volatile("" ::: "memory");  // lanes read what others have written; LDS serves a wave in order
                    const uint32_t winner = *claim;
                    const float so_far = sums[coord];  // requested together; who does not win reads it again
                    const bool go = add && winner == (uint32_t)lane;
                    if (go) {
                        sums[coord] = fmaf(coef, v, so_far);
                        *claim = 0xFFFFFFFFu;
                    }
                    asm volatile("" ::: "memory");
                    add = add && !go;
                }
            }
            if (__any(valid && (int)worker >= i)) break;  // the rest of the chunk is for later fills
#pragma unroll
            for (int u = 0; u + 1 < kChunksAhead; ++u) rec[u] = rec[u + 1];
            ptr += kWave;
            rec[kChunksAhead - 1] = record(ptr + (kChunksAhead - 1) * kWave, count);
        }
        __syncthreads();
        const bool more = i < a.n;
        uint32_t s_next = my_signs[8 * (first + wave < i ? first + wave : i - 1)];
        WorkerQ w_next = load_uniform(wq + (first + wave < i ? first + wave : i - 1));
        for (int j = first + wave; j < i; j += kQuantWaves) {
            const WorkerQ w = w_next;
            w_next = load_uniform(wq + (j + kQuantWaves < i ? j + kQuantWaves : i - 1));
            uint32_t* part = lds_stage + __builtin_amdgcn_readfirstlane((int)table[j].w);
            const uint32_t s = s_next;
            s_next = my_signs[8 * (j + kQuantWaves < i ? j + kQuantWaves : i - 1)];
            const int b = (int)w.bits;
            const __amdgpu_buffer_rsrc_t out = uniform_buffer((const char*)w.codes + (uint64_t)wg * (uint64_t)(32 * kQuantWaves * b), 16 * b * wg_groups);
            store_worker_any<2, 16>(b, part, s, lane, more, out);
        }
        if (more) __syncthreads();  // the area is reused by the next fill
    }
    if constexpr (FUSE) {
        if (has_block) {
            const int64_t left = a.d - base - 4 * lane;
            asm volatile("" ::: "memory");  // lanes read what others have written
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
                        out.resolve_bits, sk};
    const dim3 g((unsigned)((d + 1023) / 1024)), b(kQuantThreads);
    if (out.resolve_bits < 1 || out.resolve_bits > resolve_limit(n, ghat != nullptr, g.x)) return hipErrorInvalidValue;
    const unsigned lds = resolve_lds_bytes(n, out.resolve_bits, ghat != nullptr);
    if (ghat) hipLaunchKernelGGL((k_resolve<true>), g, b, lds, stream, ws.wq, a);
    else hipLaunchKernelGGL((k_resolve<false>), g, b, lds, stream, ws.wq, a);
    return hipGetLastError();
}

}  // namespace agc
