// How a wave of sconv_flat_mc_kernel walks its stream of records.  Apart from the kernel so that a host program walks the packed
// streams by the same lines (tests/host/flat_mc_check.cpp).
#pragma once

#ifdef __HIPCC__
#define SCONV_MC_WALK __host__ __device__ __attribute__((always_inline)) inline
#else
#define SCONV_MC_WALK inline
#endif

namespace sconv {

// Byte of the stream, counted from the wave's first block, at which block b begins (seg: first record and steps of each block of
// the unit).  A block in which the unit has no weights has no record: what stands there is the next block's first, or the spare one.
template <class Seg>
SCONV_MC_WALK int mc_block_at(const Seg &seg, int b, int b_first, int record_bytes) { return (seg[2 * b] - seg[2 * b_first]) * record_bytes; }

// The steps of one block; r0 holds the record that stands at the block's beginning.  load(r) takes the stream's next record;
// the steps take their own record and the `off` of the one that follows (some record's, if none follows), shared ones first.
// flush(steps left of the block) follows after six or seven steps, counted from block to block in `since`.
template <class Record, class Load, class Shared, class Private, class Flush>
SCONV_MC_WALK void mc_walk_block(Record &r0, int n_shared, int n_private, int &since, Load load, Shared shared, Private own, Flush flush)
{
    Record r1;
    r1.off = r0.off;                     // (a block of one step loads no other record, and its step reads LDS there)
    int left = n_shared + n_private;     // steps of this block still to come, this one included
    auto due = [&](int steps) __attribute__((always_inline)) {
        since += steps;
        if (since >= 6) {
            flush(left);
            since = 0;
        }
    };
    auto run = [&](int n, auto step) __attribute__((always_inline)) {
        auto one = [&](const Record &cur, Record &next) __attribute__((always_inline)) {
            if (--left) load(next);
            step(cur, next);
        };
        int i = 0;
        for (; i + 1 < n; i += 2) {
            one(r0, r1);
            one(r1, r0);
            due(2);
        }
        if (i < n) {
            one(r0, r1);
            r0 = r1;
            due(1);
        }
    };
    run(n_shared, shared);
    run(n_private, own);
}

} // namespace sconv
