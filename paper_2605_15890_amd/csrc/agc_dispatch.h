// Rules that choose between the forms of a kernel, by sizes alone.  No HIP in here: the rules are also
// compiled and checked without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace agc {

// Vectors short enough that a block's workers are shared among the four waves of a workgroup
// (k_scale_pass_parts, k_quantize<.., PARTS>).  A wave that walks over all workers alone on its SIMD mostly waits
// for itself; four waves per block hide that as long as the chip has room for them, and lose to the long form
// (four blocks per workgroup, every row read once) once it is full.  With one or two workers there is nothing to
// share.  The windows of vectors that end inside a block have lines further out (up to them the parts are still the faster
// form: W = 4, 32 workers x 196 001 33 and 39 us in the long form; W = 8, 32 x 98 001 31 and 45; 64 x 131 001 bucket-wise 51 and
// 55); a cyclic band has the same for all, us beyond its line in parts | long: max-abs 64 x 327 681 73 | 63, 64 x 500 000 93 | 67,
// 32 x 393 000 44 | 37;  Euclidean 64 x 500 000 100 | 69;  bucket-wise 64 x 500 000 77 | 51.
//   band   > 0: cyclic band of that width, -W: window driver, 0: gather driver
//   norm   Euclidean scale;  bucket: bucket-wise scales (no scale pass)
// Measured: time of a whole step in the long form over that in this one, ten steps in a graph, 6000 shapes of
// 3..256 workers.  Largest and smallest up to the line | beyond it:
//   band    4-7 workers           1.26 .. 0.99 | 262144 coordinates 1.07 .. 0.93
//           8 and more            2.09 .. 1.00 | 393216: 0.99 .. 0.77, 524288: 0.91 .. 0.65
// (tenth percentile and median up to the line | beyond it)
//   window, W <= 4                whole, 4-15 workers 0.97 and 1.08 | 0.93 and 1.00;  16-47 1.08 and 1.21 | 0.93 and
//           1.02;  48 and more 1.15 and 1.45 | 1.05 and 1.2;  ending inside, 16 and more 1.25 and 1.6 | 0.96 and 1.1
//   window, W = 8                 a part starts up to a ring of ten rows early, much of its share when rows are few,
//           and where there are more rows than workers the workers are not what takes the time:
//           whole, k <= n 1.05 and 1.15 | 0.97 and 1.0;  k <= 1.6 n 1.03 and 1.13 | 0.91 and 0.97;  k <= 2.2 n 1.0 and
//           1.12 | 0.95 and 1.0;  more 0.98 and 1.1 | 0.87 and 0.98;  64 and more 1.0 and 1.2 | 0.9 and 1.1;
//           ending inside, 16-31 1.05 and 1.3 | 0.82 and 0.95;  32 and more 1.2 and 1.5 | 0.95 and 1.2;  96 and more
//           (their codes need several fills of the staging area in the long form) 1.1 and 1.4
// (largest and smallest)
//   gather  3 and more            3.57 .. 1.00 | 393216 with fewer than sixteen workers 1.63 .. 0.82
//           16 and more, partitions with two holders 1.62 .. 0.98 | 786432 1.2 .. 0.94 (bucket-wise 524288 0.92);
//           four: 1.28 .. 1.02 | 1048576 1.05 .. 0.90;  eight: 1.48 .. 1.00
inline bool use_parts(int64_t d, int n, int k, int nnz, int band, bool norm, bool bucket)
{
    const int64_t blocks = (d + 255) / 256;
    const bool ragged = d % 256 != 0;
    if (n < 4) return n == 3 && blocks <= 256;
    if (band > 0) {
        return blocks <= (n < 8 || (norm && !bucket) ? 768 : 1024);
    }
    if (band < 0 && band >= -4) {
        if (n >= 96 || (n >= 32 && ragged)) return blocks <= 1024;
        if (n >= 48) return blocks <= 768;
        if (bucket) return blocks <= (n < 16 ? 512 : 768);
        if (n >= 16) return blocks <= (ragged ? 768 : 384);
        return blocks <= (norm ? 192 : 384);
    }
    if (band < 0) {
        const int rows = 10 * k / n;  // per ten workers; k <= 65536
        if (n >= 96 && (bucket || ragged || rows > 16)) return blocks <= 1024;
        if (bucket) {
            if (n >= 64 || (ragged && n >= 16)) return blocks <= 512;
            return blocks <= (rows <= 16 ? 512 : n >= 16 ? 192 : 64);
        }
        if (ragged && n >= 16) return blocks <= (n < 32 ? 256 : 512);
        if (n >= 64) return blocks <= 384;
        if (rows <= 10) return blocks <= 384;
        if (rows <= 16) return blocks <= (n < 32 ? 192 : 64);
        return blocks <= (ragged || rows <= 22 ? 64 : 32);
    }
    const int64_t held = nnz / k;  // workers per partition
    if (n >= 16 && held >= 8) return blocks <= 4096;
    if (n >= 16 && (held >= 4 || (held >= 2 && n >= 128))) return blocks <= (bucket && n < 128 ? 2048 : 3072);
    if (n >= 16 && held >= 2) return blocks <= (bucket && n < 48 ? 1536 : 2048);
    return blocks <= 1024;
}

// The quantize pass of long vectors: the group of four blocks that its first workgroup takes; the others follow
// upwards and wrap around.  The codes of the block that the vector ends in leave in pieces that do not fill their lines and
// are masked lane by lane, so it takes longer than the others: it is not the last to start.  With no more groups than
// the chip holds at once (four workgroups on each of 256 compute units) all start together and the order is left alone.
// Whole step, upwards from 0 | from 64 groups before the end, three runs each, us: 128 workers x 5 400 001 1096-1100 |
// 1090-1093;  64 x 25 600 001, 64 x 2 000 003, 50 x 5 400 003, 32 x 11 700 003, 4 x 25 600 003 within the runs' difference (1 %).
// Vectors of whole blocks take the same time from any group (32 x 11 700 224 521 | 522 us), so nothing of G that the
// scale pass left in the memory-side cache is gained by the order.
constexpr int64_t kChipGroups = 4 * 256;
constexpr unsigned kEarlyGroups = 64;
inline unsigned first_group(int64_t d, unsigned groups)
{
    return d % 256 != 0 && groups > kChipGroups ? groups - kEarlyGroups : 0u;
}

// One read of G (agc_sketch.h): records a block has room for.  As many as leave four workgroups of a compute unit's 160 KB of
// LDS (three and two with more workers, whose partial sums and signs take room themselves), and no more than an eighth of
// the block's coded elements, which as records of eight bytes each, written and read, move half of a second read of G.
// LDS is handed out in units of 1280 bytes: at 53 760 bytes three workgroups of 256 threads run on a compute unit, at 53 764 two
// (768 of them 358 and 673 us).  Whole steps with 53 * 1024 bytes | 42 units, us: 128 workers x 4 M 617 | 566, 100 x 4 M
// 565 | 512, 144 x 4 M 717 | 657, 160 x 3 M 623 | 573, 128 x 8 M six bits 1647 | 1642.
inline int sketch_cap(int n)
{
    const int budget = n <= 96 ? 40 * 1024 : n <= 160 ? 42 * 1280 : 64 * 1024;
    const int room = (budget - 32 * n - 4096 * ((n + 31) / 32)) / 32;
    const int cap = room < 32 * n ? room : 32 * n;
    return cap / 2 * 2;
}

// Records of a whole vector with levels 0..L_i, `levels` the sum of the L_i: its magnitudes sum to at most sqrt(d) times its
// norm, and the sketch knows 0.7 of the norm (Gaussian values: 0.8 of this).
inline double sketch_records(int64_t d, double levels) { return levels / 0.7 * __builtin_sqrt((double)d); }

// Whether one read of G and the small kernels around it are faster than two reads.  Microseconds saved, fitted to whole
// steps of 1126 shapes (4..64 workers, 15..250 M elements, three to eight bits) with Gaussian, heavy-tailed and layered values:
// 0.58 of one for every million elements of G that are not read again, less nine for three more launches, 2.8 for every
// million coordinates (signs and tables by groups of blocks) and six for every million records.
// Two reads | one, us (and the fit's gain), codes made as now, faster than when it was fitted: cyclic, 4 bits 32 x 11.7 M 570 | 383 (169);
// 3 bits 64 x 25.6 M 2390 | 1468 (861), 64 x 1 M 112 | 88 (24), 32 x 1 M 63 | 57 (7), 32 x 500 000 43 | 46 (-2), 16 x 2 M 69 | 64 (3),
// 8 x 4 M 70 | 72 (-2);  6 bits 50 x 5.4 M 435 | 324 (26), 16 x 2 M 70 | 73 (-2);  8 bits 64 x 5.4 M heavy tails 567 | 550, alike 568 | 722
// (-18), 4 x 25.6 M 217 | 253 (-43).
// A block of average magnitudes may fill three quarters of its room; the rest take k_quantize, and where the norm lies in a few
// layers, fuller ones do too.  That second pass costs the latency of a wave that walks over all workers and rows however
// few blocks it has; with sixty layers of magnitudes up to 1000 apart it was needed at 1 % of the shapes with up to 0.2 of the
// room in use on average, at 31 % with 0.25-0.3 and at 84 % with 0.3-0.4.  Without its price 46 of 1886 accepted steps were
// slower than with two reads, cyclic 59 x 700 353 115 | 149, window 59 x 965 376 138 | 165, gathered 48 of 123 partitions x
// 359 951 164 | 211; with it five of 1671, by up to 3 %.  The gather driver's times vary more than the fit knows,
// and its blocks that share their workers among waves gain nothing (64 x 300 000 79 | 112).
inline bool use_sketch(int64_t d, int n, int k, double levels, bool gather, bool parts, int cap)
{
    const double m = 1e-6 * (double)d, records = sketch_records(d, levels);
    const double full = 256.0 * records / ((double)cap * (double)d);
    if ((gather && parts) || full > 0.75) return false;
    const double again = full > 0.2 ? (gather ? 0.5 : 0.25) * (n + k) : 0.0;
    return (0.58 * k - 2.8) * m - 9.0 - 6e-6 * records - again > (gather ? 20.0 : 2.0);
}

// One read of G for the largest magnitude (k_sketch_max).  Records a block has room for: half as many bytes, written and read, as
// a second read of its rows, and no more than half of its coded elements, rounded up to halves of the ring that they wait in.
inline int sketch_max_cap(int n, int k)
{
    const int room = 32 * k < 128 * n ? 32 * k : 128 * n;
    return (room + 255) / 256 * 256;
}
// G of 4 GB and more, where what it takes to find out is little: the sample, its bounds and kernels that have nothing to do, 20-60 us.
// Whether one read saves anything depends on the values, and the sample decides that on the device (sketch_max_limit); the wider the
// codes, the fewer the values with which it does.  Whole steps, two reads | one, us: heavy tails (t, three degrees), three bits on
// average, cyclic 64 workers x 25.6 M 2320 | 1623, 40 x 27 M 1512 | 1095, 24 x 45 M 1507 | 1129, 12 x 90 M 1619 | 1444;  windows, 10 workers
// and 30 partitions x 36 M 1428 | 923, 64 x 25.6 M 2305 | 1751;  gathered 64 x 25.6 M 6900 | 3745;  sixty layers of magnitudes up to
// 1000 apart 64 x 25.6 M 2310 | 2057, 40 x 27 M 1520 | 1380, 24 x 45 M 1513 | 1437.  Values that are alike everywhere, which the sample
// refuses: 64 x 25.6 M 2282 | 2303 and on other cards 2344 | 2372, 2324 | 2387;  40 x 27 M 1518 | 1565, 10 of 30 x 36 M 1428 | 1457,
// 12 x 90 M 1614 | 1663.  Below the line heavy tails would gain as much (64 x 12.8 M 1196 | 888, 64 x 6.4 M 616 | 492, 32 x 25.6 M
// 1168 | 845, 16 x 25.6 M 620 | 531) and alike values lose more (64 x 6.4 M 607 | 627, 10 of 30 x 5.4 M 247 | 265).  Eight workers gain
// nothing (8 x 25.6 M 330 | 344).  Five bits, 64 x 25.6 M, forced: heavy tails 2451 | 2241, with layers 2455 | 1916;  six 2522 | 2743, 2523 | 2177.
// The vector fills the chip several times over, since the bounds rise with what has been read.  With more than 128 workers too few
// workgroups fit a compute unit: 128 x 8.5 M 1641 | 1302, 256 x 5.3 M 2099 | 2003.
inline bool use_sketch_max(int64_t d, int n, int k, double levels)
{
    return k >= 12 && n <= 128 && d >= 20480 * 256 && (int64_t)k * d >= (int64_t)1 << 30 && levels <= 16.0 * n;
}
// What the sampled blocks may cost for the sketch to be made (k_sketch_bounds_max), in units of 1 / kReadCost of a second read of a
// block's rows.  A block that overflows costs all of it, any other half of the part of its room that it fills (records are written and
// read).  Fitted to both forms' times of 198 steps, 10-64 workers, 12-64 partitions, 4.3-6.5 GB of G, two to four bits: of those that
// are taken one is 2 % slower than with two reads, the others at most 1 %.  Two reads | one, us, and cost (line): cyclic 64 x 25.6 M, heavy tails, two to
// four bits 2313 | 1463 0.07 (0.44), 2363 | 1648 0.13, 2416 | 1935 0.31;  layers 2321 | 1772 0.12, 2361 | 2087 0.28, 2417 | 2377 0.43;
// alike, two bits 2307 | 3249 1;  12 x 90 M, two bits, heavy tails 1627 | 1384 0.08 (0.17), Laplace 1626 | 1712 0.17 and alike
// 1628 | 1954 0.22, whose blocks do not overflow;  16 x 68 M, one in a hundred values the largest, two bits, 0.5, 0.7, 0.85, 0.95 and 1.05
// rooms of records 1573 | 1505 0.25 (0.25), 1574 | 1560 0.35, 1589 | 1652 0.43, 1591 | 1862 0.6, 1595 | 2846 1.
constexpr uint32_t kReadCost = 64;
inline uint32_t sketch_max_limit(int k, int samples)
{
    const double share = 0.5 - 4.0 / k;
    return share > 0.0 ? (uint32_t)(share * kReadCost * samples) : 0u;
}

// Bytes of the sketch's two large arrays, signs and records: 0.97 GB at 64 workers x 25.6 M, 15 % of G there and up to half of
// G for four workers;  for the largest magnitude 1.9 GB, 28 %.
inline int64_t sketch_bytes(int n, int64_t d, int cap)
{
    return (d + 255) / 256 * ((int64_t)((n + 31) / 32) * 1024 + 8 * (int64_t)cap);
}
inline int64_t sketch_bytes(int n, int64_t d) { return sketch_bytes(n, d, sketch_cap(n)); }
// A context takes them only beside a G that leaves half of the card to the rest of the program (the context may be made
// first), and no more than an eighth of what is free: a program that fills the card keeps the form with two reads and the
// memory that it had.
inline bool sketch_fits(int n, int k, int64_t d, size_t free_bytes, size_t total_bytes, int cap)
{
    const double bytes = (double)sketch_bytes(n, d, cap);
    return bytes + 4.0 * k * (double)d <= 0.5 * (double)total_bytes && bytes <= 0.125 * (double)free_bytes;
}
inline bool sketch_fits(int n, int k, int64_t d, size_t free_bytes, size_t total_bytes)
{
    return sketch_fits(n, k, d, free_bytes, total_bytes, sketch_cap(n));
}

// The blocks that the bounds of the scales are estimated from: one of each of `samples` runs of equal length (up to one
// block), drawn anew for every step.  At a fixed distance, up to 8.4 M coordinates a power of two, the sample saw the same columns of
// every row of a gradient made of matrices, in every step: with the first 256 of 4096, 8192 or 16 384 columns 20 times as
// large the bounds did not hold, at a twentieth they lay so low that no block had room for its records, and a step took 9-15 and
// 10-34 % longer than with two reads (50 workers x 5.4 M, 64 x 5.4 M, 32 x 2 M, 64 x 1 M).
// One block in 32, and at most 512.  The bound leaves the two largest out, so of a norm that lies in a 32nd of the vector one
// block in 64 saw nothing at 1 M coordinates: 64 x 1 M 131 us with two reads, 139 with one block in 64, 116 with one in 32;
// 32 x 2 M 125 | 122 | 106.  Values that are alike everywhere 108.4 | 108.4 and 108.8 | 109.0, one block in 16 110.5 and 111.8.
constexpr int kMaxSamples = 512;
inline int sample_count(int64_t nblocks)
{
    return nblocks < 32 ? 1 : nblocks / 32 < kMaxSamples ? (int)(nblocks / 32) : kMaxSamples;
}
struct SampleRuns {
    int64_t length, longer;  // blocks of a run; the first `longer` runs have one more
    uint64_t salt;
};
// SplitMix64's output function (Steele, Lea, Flood 2014)
constexpr uint64_t mix64(uint64_t x)
{
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
inline SampleRuns sample_runs(int64_t nblocks, int samples, uint64_t seed, uint64_t step)
{
    return SampleRuns{nblocks / samples, nblocks % samples,
                      mix64(seed + mix64(step + 0x9E3779B97F4A7C15ull))};
}
constexpr int64_t sample_block(const SampleRuns& r, int64_t e)  // device too
{
    const int64_t first = e * r.length + (e < r.longer ? e : r.longer);
    const uint64_t length = (uint64_t)(r.length + (e < r.longer ? 1 : 0));  // < 2^32
    return first + (int64_t)(((mix64(r.salt + 0x9E3779B97F4A7C15ull * (uint64_t)e) >> 32) * length) >> 32);
}

// Workgroups of the decode pass that a compute unit holds: six, which was measured to be best with one scale per
// vector (walking over the tiles: five 0.162, four 0.166 against 0.148 ms for 64 workers x 25.6 M), or as many as
// 160 KB of LDS has room for beside the weights of bucket- and layer-wise scales: five, four with two tracks and
// layers.
constexpr int decode_per_cu(unsigned lds_bytes)
{
    return 160 * 1024 / lds_bytes < 6 ? (int)(160 * 1024 / lds_bytes) : 6;
}

// Workgroups of the decode pass.  As many as the chip holds, which then walk over the tiles and fetch the next
// tile's first chunk during the last of this one; more would start when the first ones have finished everything
// (six per compute unit where five fit: 64 workers, layer-wise, 5.4 M 72 | 66 us, 10 workers 25.6 M 75 | 69).  But
// with four chunks and more to a tile, that prefetch is a small part of the work, and from two tiles a workgroup on
// the uneven rest of the tiles costs more than it saves: there one workgroup per tile, handed out as they finish
// (128 workers, 25.6 M, walking | one per tile: 401 | 372 us, layer-wise 463 | 421, two tracks 481 | 442; two
// chunks: 10 workers 64 | 73).
inline int64_t decode_groups(int64_t tiles, int chunks, int per_cu)
{
    const int64_t resident = 256 * (int64_t)per_cu;
    if (chunks >= 4 && 4 * tiles >= 7 * resident) return tiles;
    return tiles < resident ? tiles : resident;
}

// Decode of one track without chunks (k_decode_direct): one or two workers, where most of a chunk would be fetched
// twice to fill it, and up to four on vectors so long that the stores of the estimate decide.  Whole decode with
// eight coordinates per lane | direct, us: 1 worker, 4 bits, 4096 coordinates 5.1 | 4.6, 500 000 6.2 | 5.9,
// 25.6 M 44 | 41;
// 2 workers, 4 bits each, 500 000 6.6 | 6.4;  3 workers 500 000 6.9 | 7.2, 25.6 M 47 | 46, 60 M 103 | 96;  4 workers
// 60 M 105 | 99.
inline bool decode_is_direct(int n_arrived, int64_t d)
{
    return n_arrived <= (d >= ((int64_t)1 << 25) ? 4 : 2);
}

// Coordinates per lane of the decode pass.  Sixteen halve the per-worker overhead of eight; eight double the number
// of waves, and with a chunk's worth of codes the overhead is little.  us with eight | sixteen: 64 workers, 192 bits,
// one scale: 2.1 M 36 | 41, 4 M 52 | 55, 5.4 M 70 | 70, 8 M 93 | 89, 25.6 M 183 | 148;  bucket-wise 3.5 M 54 | 58,
// 4 M 63 | 59, 8 M 113 | 93;  8 workers, 32 bits: 5.4 M 17.6 | 22, 25.6 M 53 | 63;  16 workers, 48 bits, 25.6 M
// 82 | 79.  The two-track decode holds twice the accumulators and is faster with eight throughout (50 workers, four
// bits, 5.4 M coordinates, with the update: 79.5 us with eight, 86.8 with sixteen; 24 workers, 25.6 M: 260 and 285).
//   many_scales: bucket- or layer-wise;  sum_bits: of the workers that arrived
inline int decode_coords(int64_t d, bool two, bool many_scales, int sum_bits)
{
    if (two || sum_bits <= 40) return 8;
    return d >= (many_scales ? (int64_t)15 << 18 : (int64_t)5 << 20) ? 16 : 8;
}

// Least squares: samples side by side in a row slot (k_ls_resident), for rows of at most 1024 features.  The widest
// fold keeps all lanes busy; but a block is then 32 * fold samples whether they exist or not, so the fold is no wider
// than a partition fills.  Up to 4096 samples in all (128 workgroups of 32) nothing but the time of one block
// counts, and that is shortest without.  Features, partitions, samples per partition: without | with the widest, us:
// 128, 32, 16 7.0 | 9.4, 128, 1, 4096 9.2 | 9.2, 128, 16, 512 10.6 | 8.9, 128, 128, 64 9.9 | 9.6 (two 8.3),
// 1024, 4, 256 8.1 | 9.2, 1024, 128, 48 10.3 | 11.3, 512, 4, 16384 28 | 17.
// The sums of a block without fold are chains of 32 samples, with it shorter ones: relative error against binary64
// 0.6e-7 to 1.5e-7 without, 0.6e-7 to 1.3e-7 with the widest, at sizes where the rule takes none or a smaller one.
inline int ls_fold(int64_t n_rows, int64_t rows_per_part, int n_feat)
{
    if (n_rows <= 4096) return 1;
    int fold = n_feat <= 128 ? 16 : n_feat <= 256 ? 8 : n_feat <= 512 ? 4 : n_feat <= 1024 ? 2 : 1;
    while (fold > 1 && 32 * fold > rows_per_part) fold /= 2;
    return fold;
}

// Least squares: few enough parts of a partition (one per workgroup) for one thread per feature in their sum.  Many
// parts are shared by eight threads per feature, which hides the memory's latency (65536 x 512 samples x features,
// 512 parts 18 us, one thread 34); up to sixteen parts one thread requests all of them together, and eight would only
// be eight times as many workgroups (2^17 x 8192, one part: 387 us, now 346; 65536 x 4096, 8 parts 92, now 87).
constexpr bool ls_reduce_few(int wg_per_part) { return wg_per_part <= 16; }

}  // namespace agc
