// Launch interface between the C ABI (agc_api.cpp) and the gfx950 kernels (agc_kernels.hip).
// Plain structs only; every pointer is a device pointer unless it sits inside an argument
// block, which travels to the GPU as kernel arguments.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "agc_dispatch.h"
#include "agc_stream.h"

namespace agc {

constexpr int kArgWorkers = 256;

// Row i of a monotone-interval code as one 64-byte record, so that a kernel reads a worker's
// structure with scalar loads whose address depends on i alone (no row_ptr -> col -> val chain).
// Record n is a sentinel whose lo matches no row.
struct WindowRec {
    int lo;               // first column of the run
    int len;              // 1..8 stored entries
    int pad[6];
    float val[8];         // the entries in stored order; unused ones are 0 and never read
};
static_assert(sizeof(WindowRec) == 64, "one record is 64 bytes");

struct CodeDev {          // the code matrix B on the device
    const int* row_ptr;   // [n+1]
    const int* col;       // [nnz]
    const float* val;     // [nnz]
    int band;             // 0: generic CSR; s>0: cyclic band with s entries per row; -W: monotone intervals
    const WindowRec* win; // [n+1], monotone-interval codes only (else null)
    bool parts;           // use_parts() of this code
    const StreamRec* stream;  // [nnz+1], codes that stream_records takes (else null)
};

// what the quantize pass needs to know about worker i, read with one scalar 32-byte load
struct WorkerQ {
    float inv16;          // L_i * 2^16 / scale_i (2^15 / scale_i for a one-bit worker); with bucket-wise
                          // scales the numerator alone, the division happens per block
    uint32_t bits;
    void* codes;          // packed stream of the worker
    // fused quantize+decode pass only: the decode weight of worker i (w_i * scale_i / L_i; with
    // bucket-wise scales w_i / L_i) and whether it arrived
    float coef;
    uint32_t arrived;
    // where the worker's codes wait in the workgroup's LDS staging area before they leave as whole
    // 128-byte lines: first 16-byte piece of the worker (a workgroup stages 8 * bits pieces per
    // worker: four blocks of 2 * bits), and whether the area is written out after this worker
    uint32_t stage_piece;
    uint32_t flush;
};
static_assert(sizeof(WorkerQ) == 32, "one record is two 16-byte scalar loads");

// The staging area of a workgroup holds the codes of consecutive workers whose bit-widths sum to
// at most a cap (8 * cap pieces of 16 bytes); workers beyond that start a new fill.  Up to the limit the
// codes of all workers wait in one fill, which leaves the loop over the workers free of stores.
// The limit is what leaves room for four workgroups per compute unit.  50 workers with 300 bits in all: one
// fill 478 us, two fills (a limit of 256) 493 us for the whole encode; 64 workers with 384 bits: two fills at
// four workgroups 644-675 us, one fill at three workgroups 650-678 us.
constexpr int kStageLds = 160 * 1024 / 4;
constexpr int kStageBits = (kStageLds - 16) / 128;  // 319
// the same beside the bucket-wise scales of four blocks
inline int stage_limit(int n, bool bucket) { return bucket ? (kStageLds - 16 - 16 * n) / 128 : kStageBits; }

// All fills about equally full: the area, and with it the LDS of a workgroup, is as small as the number of
// fills allows.  A fill that is closed because a worker of up to 16 bits does not fit holds more than
// cap - 16 bits.
inline int stage_cap(const uint8_t* bits, int n, int limit)
{
    int sum = 0;
    for (int j = 0; j < n; ++j) sum += bits[j];
    const int fills = (sum + limit - 1) / limit;
    if (fills <= 1) return limit;
    const int cap = (sum + fills - 1) / fills + 15;
    return cap < limit ? cap : limit;
}
// Places the workers in the staging area (host side): start[i] = sum of the bit-widths staged
// before worker i in its fill; a fill ends before the worker that would overflow it, and that worker starts
// the next one at 0.  Returns the number of fills; *most is the fullest one, in bits.
inline int stage_starts(const uint8_t* bits, int n, int limit, uint16_t* start, int* most)
{
    const int cap = stage_cap(bits, n, limit);
    int acc = 0, fills = n > 0 ? 1 : 0;
    *most = 0;
    for (int j = 0; j < n; ++j) {
        if (acc + bits[j] > cap) {
            acc = 0;
            ++fills;
        }
        start[j] = (uint16_t)acc;
        acc += bits[j];
        if (acc > *most) *most = acc;
    }
    return fills;
}

// The same area of k_resolve, in fills of its own.  LDS of a workgroup: the area in pieces of 16 bytes, a record of 16 bytes and four
// blocks' signs for every worker, and with the estimate a sum and a claim for each of its 1024 coordinates.
constexpr int resolve_pieces(int stage_bits) { return 8 * stage_bits + 1; }
constexpr unsigned resolve_lds_bytes(int n, int stage_bits, bool fuse)
{
    return 16u * (unsigned)(resolve_pieces(stage_bits) + n) + 16u * (unsigned)(8 * n + 8) + (fuse ? 8192u : 0u);
}
// Bits of a fill: what leaves room for six workgroups on a compute unit, which is what its registers allow too (k_resolve, us,
// five | six | seven at 64 workers x 25.6 M: heavy tails, largest magnitude 404 | 374 | 425, Euclidean 245 | 232 | 282;  50 x 5.4 M,
// 300 bits, without estimate 86 | 84 | 78), but no less than 48, where that many do not fit.  Vectors of which no more than four or
// five come to a compute unit have larger fills, hence fewer, one after the other in the chain of a workgroup.  Whole steps, Euclidean,
// three bits, room for six | for what there are, us: 64 x 600 000 79.2 | 76.3, 64 x 1 M 90.4 | 88.0, 64 x 1.2 M 108.3 | 106.0, 128 x 700 000
// 131.4 | 123.7;  five bits 64 x 1 M 105.5 | 100.4, 64 x 1.2 M 122.7 | 118.0.
constexpr int kResolveWgs = 6;
inline int resolve_limit(int n, bool fuse, int64_t groups)
{
    const int per_cu = groups <= 4 * 256 ? 4 : groups <= 5 * 256 ? 5 : kResolveWgs;
    const int room = 160 * 1024 / per_cu / 1280 * 1280, rest = (int)resolve_lds_bytes(n, 0, fuse);
    const int bits = (room - rest) / 128;
    return bits < 48 ? 48 : bits;
}

// Short vectors (use_parts): the codes of one block wait in LDS in a single fill, 32 bytes per bit of width: all
// 256 workers at four bits or 64 at sixteen.
constexpr int kPartBits = 1024;

// ---- tables of the decode pass.  A tile of the vector is 256 * COORDS coordinates; a worker's part of it
// is `bits` units of 32 * COORDS contiguous bytes.  Units of consecutive workers, whole workers only, fill
// chunks of kDecChunkBytes, which is what a workgroup fetches at a time.
constexpr int kDecChunkBytes = 12288;

struct DecWorker {        // one arrived worker; read with scalar loads (k_decode: the first half)
    float coef;           // w_i * scale_i / L_i (bucket-wise scales: w_i / L_i; layer-wise: unused)
    float coef2;          // the same with the second decoding vector
    uint32_t width;       // 1 << bits; 1 for two bits and weights that can be halved exactly
    uint32_t pos;         // its first unit within its chunk
    uint32_t worker;
    uint32_t bits;
    const char* codes;    // its stream
};
static_assert(sizeof(DecWorker) == 32, "one record is two 16-byte scalar loads");

struct DecUnit {
    const char* codes;    // the unit of tile 0
    uint32_t tile_pieces; // 16-byte pieces from one tile to the next
    uint32_t pieces;      // 16-byte pieces from here to the end of the stream, >= 1
};
static_assert(sizeof(DecUnit) == 16, "one record is one 16-byte load");

struct DecodeTables {
    DecWorker* workers;
    DecUnit* units;
    int* chunk_first;     // [n_chunks + 1]
};

// Most units the chunks of n workers have room for: a chunk of 24 (48) units holds at least one worker, and
// is closed when the next one of up to 16 units does not fit, i.e. with at least 33 of the 48 in use.
// So there are at most n chunks of 24, or 16n/33 + 1 chunks of 48.
constexpr int64_t decode_units(int n) { return 24 * (int64_t)n + 48; }
constexpr size_t decode_table_bytes(int n)
{
    return sizeof(DecWorker) * (size_t)n + sizeof(DecUnit) * (size_t)decode_units(n) + sizeof(int) * ((size_t)n + 2);
}

struct Workspace {
    uint32_t* part_max;   // [max_rows][n] running max |f_i| as bit patterns, all zero between steps (max-abs scale)
    int max_rows;         // kMaxSlots, or n_layers * kLayerSub if that is more
    double* part_sq;      // [nseg][n]   per-segment sum of squares             (Euclidean scale)
    double* group_sq;     // [n][ngroup] (layer-wise: [n][ngroup_layers])
    WorkerQ* wq;          // [n]  written by the scale finalize
    void* dec;            // decode_table_bytes(n) bytes: tables of the arrived workers, written by the decode prologue
    int64_t nseg, ngroup;
    // layer-wise scales (n_layers > 0): the layer of every 256-coordinate block, and
    // the decode weights w_i * scale_il / L_i (and v_i * ...) of the arrived workers, [layer][slot].
    // wq then holds one table per layer, [layer][n].
    const uint8_t* block_layer;  // [ceil(d/256)]
    int n_layers;
    // Euclidean scale per layer: the summation tree starts anew in every layer, so the segments
    // (up to four blocks) are counted from each layer's first block
    const int* seg_first;        // [nseg_layers] first block of the segment
    const uint8_t* seg_blocks;   // [nseg_layers] its number of blocks, 1..4
    const int* group_seg;        // [ngroup_layers + 1] first segment of every group (64 of one layer at most)
    const int* layer_group;      // [n_layers + 1] first group of every layer
    int64_t nseg_layers, ngroup_layers;
    float* coef_layer;    // [n_layers][n]
    float* coef2_layer;   // [n_layers][n]
};

// What k_sketch leaves behind of its one read of G (agc_sketch.h), and the small tables around it.
struct SketchDev {
    uint32_t* planes;     // [block][worker, up to 32 * chunks][8] signs, in the order of the coordinates; null: not available
    uint2* recs;          // [block][cap] coded values whose level depends on the scale
    int* counts;          // [4 * groups of four blocks] records of the block; -1: there were more than cap
    float* lo_scale;      // [n] lower bounds of the scales, and the largest multipliers that they leave
    float* lo_mult;       // [n]
    uint32_t* state;      // [3] not 0: a bound did not hold, or a weight is not finite, or there is no sketch;  length of the
                          // list;  largest magnitude: what the sampled blocks would cost, 0 between steps
    uint32_t limit;       // largest magnitude: above it G is read twice after all
    uint4* table;         // [n] what k_resolve needs to know of a worker: multiplier, weight, bits with 256 arrived and 512 end of a
                          // fill, first word in the staging area
    uint32_t* left;       // [groups of four blocks] list of those that k_resolve leaves to k_quantize, in any order
    int cap;              // even
    int chunks;           // ceil(n / 32)
};
// LDS of a k_sketch workgroup: [4][n] doubles, [4][chunks] KB of signs, [4][cap] records
constexpr unsigned sketch_lds_bytes(int n, int cap) { return 32u * n + 4096u * ((n + 31) / 32) + 32u * cap; }

// LDS of a k_sketch_max workgroup: for each of its waves a ring of 512 records, [chunks] KB of signs, [n] maxima and multipliers
constexpr unsigned sketch_max_lds_bytes(int n) { return 4u * (4096u + 1024u * ((n + 31) / 32) + 8u * ((n + 1) / 2 * 2)); }

constexpr int kMaxSlots = 256;  // rows of the max-abs array; a block folds into row (block mod kMaxSlots)
constexpr int kMaxLayers = 256;  // layer-wise scales: a block's layer fits a byte
constexpr int kLayerSub = 16;    // with layer-wise scales layer l owns rows l*kLayerSub .. +kLayerSub-1 of the array

struct QuantStreams {      // host arrays of the encode call
    void* codes[kArgWorkers];
    uint8_t bits[kArgWorkers];
    uint16_t stage_start[kArgWorkers];  // stage_starts() of the bit-widths
    int stage_fills, stage_bits;        // and what it returns: fills, the fullest one in bits
    uint16_t resolve_start[kArgWorkers];  // the same for the fills of k_resolve, where it runs
    int resolve_bits;
    bool parts;                         // the quantize pass shares the workers of a block among the waves
};

struct BitList {           // bit-widths as a kernel argument
    uint8_t bits[kArgWorkers];
};
inline BitList bit_list(int n, const QuantStreams& out)
{
    BitList bits;
    for (int i = 0; i < kArgWorkers; ++i) bits.bits[i] = i < n ? out.bits[i] : 0;
    return bits;
}

struct StepWeights {       // decode side of a fused step
    float w[kArgWorkers];
    uint8_t arrived[kArgWorkers];
    int fuse;              // 0: plain encode+quantize, the two arrays are ignored
};

template <int CAP>
struct QuantList {         // both as kernel arguments of the table kernels, for up to CAP workers
    void* codes[CAP];
    float w[CAP];
    uint8_t bits[CAP];
    uint16_t stage_start[CAP];
    uint8_t arrived[CAP];
    int fuse;
};

struct DecodeStreams {     // the arrived workers of a decode call, in ascending order (host side)
    int n_arrived;
    const void* codes[kArgWorkers];
    float w[kArgWorkers];
    float v[kArgWorkers];        // second decoding vector of the two-track decode (Sec. V)
    uint8_t bits[kArgWorkers];
    uint8_t worker[kArgWorkers]; // which worker it is
};

template <int CAP>
struct DecodeList {        // the same as kernel arguments of the decode's prologue, with the places in the chunks
    int n_arrived;
    int units_per_chunk;   // 0: the decode takes no chunks (k_decode_direct)
    int unit_pieces;       // 16-byte pieces of a unit
    uint32_t groups;       // 128-code groups of a stream
    const void* codes[CAP];
    float w[CAP];
    float v[CAP];
    uint8_t bits[CAP];
    uint8_t worker[CAP];
    uint8_t chunk[CAP];
    uint8_t pos[CAP];
};

// K1: partial results of every worker's scale (max-abs: running maxima in ws.part_max, per layer
// with layer-wise scales; Euclidean: per-segment sums of squares).  scale_mode: 0 Euclidean, 1 max-abs.
hipError_t launch_scale_pass(const float* G, int64_t ldg, int n, int k, int64_t d,
                             const CodeDev& code, int scale_mode, const Workspace& ws,
                             const SketchDev* sk, hipStream_t stream);
// all rows of the max-abs slot array, and the sketch's state[2] if there is one, back to zero
hipError_t launch_scale_clear_slots(int n, const Workspace& ws, uint32_t* state, hipStream_t stream);
// K1f: partials -> scales[n] and the per-worker table of the quantize pass (with layer-wise scales:
// scales[n][n_layers] and one table per layer).
// sw.fuse != 0: the quantize pass that follows also forms the estimate (ghat) from the codes it
// has just produced, in the same order and arithmetic as the decode kernel.
hipError_t launch_scale_finalize(int n, int scale_mode, const QuantStreams& out, const StepWeights& sw,
                                 const Workspace& ws, const SketchDev* sk, float* scales, hipStream_t stream);
// One read of G (Euclidean scale of the whole vector): bounds from a sample, then the sketch; it leaves the partial results
// of the scales like the scale pass.  launch_scale_finalize with the same sk checks the bounds.
hipError_t launch_sketch_bounds(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code,
                                const Workspace& ws, const SketchDev& sk, const QuantStreams& out, uint64_t seed,
                                uint64_t step, hipStream_t stream);
hipError_t launch_sketch(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code, const Workspace& ws,
                         const SketchDev& sk, uint64_t seed, uint64_t step, hipStream_t stream);
hipError_t launch_sketch_bounds_max(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code, const Workspace& ws,
                             const SketchDev& sk, const QuantStreams& out, uint64_t seed, uint64_t step, hipStream_t stream);
// One read of G for the largest magnitude of the whole vector; the scales' partial results are in the first row of ws.part_max.
hipError_t launch_sketch_max(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code, const Workspace& ws,
                             const SketchDev& sk, const QuantStreams& out, uint64_t seed, uint64_t step, hipStream_t stream);
// codes (and with ghat the estimate) of the sketch; launch_quantize with sk makes those of the groups it leaves
hipError_t launch_resolve(int n, int64_t d, const Workspace& ws, const SketchDev& sk, const QuantStreams& out, uint64_t seed,
                          uint64_t step, float* ghat, hipStream_t stream);
// K2: fused encode + stochastic quantize + bit-pack.
// ghat != nullptr: fused step (the table must have been written with sw.fuse != 0).
// out: its bit-widths size the LDS staging area (the table holds them too).
hipError_t launch_quantize(const float* G, int64_t ldg, int n, int k, int64_t d,
                           const CodeDev& code, const Workspace& ws, const QuantStreams& out, uint64_t seed,
                           uint64_t step, float* ghat, const SketchDev* sk, hipStream_t stream);
// Bucket-wise scales (one per 256-coordinate block and worker): a table prologue, then ONE pass
// over G that derives each block's scale from the block itself.  scales: n x nb, nb = ceil(d/256).
hipError_t launch_quantize_bucket(const float* G, int64_t ldg, int n, int k, int64_t d, const CodeDev& code,
                                  int scale_mode, const QuantStreams& out, const StepWeights& sw,
                                  const Workspace& ws, float* scales, uint64_t seed, uint64_t step, float* ghat,
                                  hipStream_t stream);
// K3: tables of the arrived workers (a prologue), then masked dequantize + weighted sum.
// nb = 0: one scale per worker; nb > 0: scales is n x nb, one scale per 256-coordinate bucket.
// two: the same read of the codes feeds a second weighted sum, with weights in.v, into ghat2.
hipError_t launch_decode(int n, int64_t d, const DecodeStreams& in, bool two, const float* scales, int64_t nb,
                         const Workspace& ws, float* ghat, float* ghat2, hipStream_t stream);
// The one-track decode with its tables in a fixed device array instead of a context's workspace: no
// allocation anywhere, n <= 256.  Calls on one GPU share the array.
hipError_t launch_decode_static(int64_t d, const DecodeStreams& in, const float* scales, int64_t nb, float* ghat,
                                hipStream_t stream);
// Adam update that takes its first moment from ghat and its second moment from ghat2.
hipError_t launch_adam_update(float* beta, float* m1, float* m2, const float* ghat, const float* ghat2,
                              float lr, float beta1, float beta2, float eps, float corr1, float corr2,
                              int64_t d, hipStream_t stream);

// Least-squares partial gradients G[p,:] = X_p^T (X_p w - y_p) (X bfloat16) and the descent update.
int ls_wg_per_part(int64_t n_rows, int n_feat, int k_parts);
hipError_t launch_ls_partial_gradients(const void* X, int64_t n_rows, int n_feat, const float* y,
                                       const float* w, int k_parts, float* G, int64_t ldg,
                                       float* resid, float* partial, hipStream_t stream);
hipError_t launch_gd_update(float* beta, const float* ghat, float lr, int64_t d, hipStream_t stream);

// measurement kernels (agc_debug.hip): plain streaming copy of `bytes` (multiple of 16) bytes, and
// the bare row-walk access pattern of the streaming passes (piece_bytes = 0: reads only)
hipError_t launch_calibration_copy(void* dst, const void* src, int64_t bytes, hipStream_t stream);
hipError_t launch_stream_rows(const float* G, int64_t ldg, int k, int64_t d, int piece_bytes, int wg_flush,
                              int blocks_per_wave, int waves_per_simd, int fma_per_row, void* out, hipStream_t stream);

}  // namespace agc
