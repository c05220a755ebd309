// Arithmetic of the kernels that can be run on the host as it is: plain C++ without device state, so that a test compiles
// this very code for the CPU.
#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define OOCO_HD __host__ __device__ __forceinline__
#else
#define OOCO_HD inline
#endif

namespace ooco {

// floor((a * b - c) / n) for c = 0 or 1 and a quotient below 2^30, given 1 / n to two units in its last place: the product with
// the reciprocal is off by one at most, which the exact remainder corrects.
OOCO_HD int quotient_by_reciprocal(int a, int b, int c, int n, double inv)
{
    int q = (int)(((double)a * (double)b - (double)c) * inv);
    const int64_t r = (int64_t)a * b - c - (int64_t)q * n;
    q += r < 0 ? -1 : r >= n ? 1 : 0;
    return q;
}

// The arrival counter of a split prefill tile whose parts share its merge, as one word of bytes: parts that have arrived,
// draws of a slice, parts that left without waiting any longer.  The part that arrives last takes slice 0 and the parts that
// are there draw the others.  Every part ends with one event of its own -- a draw that finds no slice, or leaving --, so the
// last event of all, which resets the word for the next call, is known by its number: nobody touches the word any more.
struct MergeWord {
    static constexpr int kSlices = 4;
    static constexpr int kArrive = 1, kDraw = 1 << 8, kLeave = 1 << 16;
    static OOCO_HD int arrivals(int w) { return w & 255; }
    static OOCO_HD int draws(int w) { return (w >> 8) & 255; }
    static OOCO_HD int leaves(int w) { return (w >> 16) & 255; }
    // w: the word that an arrival, a draw or a leave found
    static OOCO_HD bool arrived_last(int w, int nparts) { return arrivals(w) == nparts - 1; }
    static OOCO_HD int slice(int w) { return draws(w) < kSlices - 1 ? draws(w) + 1 : -1; }   // -1: none left, the part ends
    static OOCO_HD bool last_event(int w, int nparts) { return draws(w) + leaves(w) + 1 == kSlices - 1 + nparts; }
};

// The KV append's choice of workgroups: of the two (sequence, block) pairs per sequence and one per 16 rows, or of one per row, which
// is half as many where nearly all sequences have one row.  `workgroups` is the former number with all parts.
OOCO_HD bool append_by_rows(int total_q, int num_seqs, int64_t workgroups, int num_cus)
{
    return 4 * (int64_t)total_q <= 5 * (int64_t)num_seqs && workgroups > num_cus;
}

// Whether the KV append's 16-byte stores go past the caches, by the bytes of K and V that it writes (see launch_kv_append).
OOCO_HD bool append_past_caches(int total_q, int num_seqs, int64_t bytes)
{
    return bytes > 8 * (1 << 20) || (num_seqs >= 16 && total_q < 100 * (int64_t)num_seqs);
}

}  // namespace ooco
