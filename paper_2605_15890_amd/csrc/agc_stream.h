// Codes whose rows of G the worker side streams once (encode_stream): which they are, and the order of their entries.  No HIP
// in here: the records are also made and checked without a GPU.
#pragma once

#include <stdint.h>

#include <vector>

namespace agc {

// Entry of a code whose rows are long intervals, in the order in which the columns' rows of G arrive (encode_stream): columns
// ascending, workers ascending within a column.  The last one is a sentinel whose column matches no row.
struct StreamRec {
    int col;
    float val;
    int slot;             // which of the open workers: 0..kStreamSlots - 1, counted from the lowest
    int last;             // the worker's last entry: it is formed, and the others move down a slot
};
static_assert(sizeof(StreamRec) == 16, "one record is one 16-byte scalar load");
constexpr int kStreamSlots = 2;

// The entries of a code whose rows are runs of consecutive ascending columns with neither end decreasing from worker to worker,
// in the order of encode_stream, and a sentinel; empty if the code is not one, or too many workers are open at a time, or
// a column has no holder.  Every row of G is read, so rows that nobody holds would cost what the others do.  Whole steps in the
// general driver | streamed, us: ten workers with ten columns each of 5.4 M coordinates, of 91 columns (all held)
// 650 | 636, of 110 723 | 760, of 120 723 | 824, of 200 723 | 1355;  of 200 columns of 400 000 84 | 151;  two workers with forty of
// 120 columns 295 | 815.
inline std::vector<StreamRec> stream_records(int n, int k, const int32_t* row_ptr, const int32_t* col, const float* val)
{
    std::vector<StreamRec> out;
    int held = 0;  // columns 0..held-1 have a holder
    for (int i = 0; i < n; ++i) {
        const int e0 = row_ptr[i], e1 = row_ptr[i + 1];
        if (e0 == e1 || col[e0] > held) return {};
        for (int e = e0 + 1; e < e1; ++e)
            if (col[e] != col[e - 1] + 1) return {};
        if (i > 0 && (col[e0] < col[row_ptr[i - 1]] || col[e1 - 1] < col[e0 - 1])) return {};
        held = col[e1 - 1] + 1;
    }
    if (held != k) return {};
    int lowest = 0, next = 0;  // workers lowest..next-1 are open
    for (int j = 0; j < k; ++j) {
        while (next < n && col[row_ptr[next]] == j) ++next;
        const int first = lowest, end = next;
        for (int i = first; i < end; ++i) {
            if (i - lowest >= kStreamSlots) return {};
            const int e = row_ptr[i] + (j - col[row_ptr[i]]);
            const int last = e + 1 == row_ptr[i + 1];
            out.push_back(StreamRec{j, val[e], i - lowest, last});
            lowest += last;
        }
    }
    out.push_back(StreamRec{INT32_MAX, 0.f, 0, 0});
    return out;
}

}  // namespace agc
