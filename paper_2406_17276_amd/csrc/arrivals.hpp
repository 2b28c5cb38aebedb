// One-shot build as one launch: how the workgroup that drafts a sequence learns which rows are there, and who drafts where it
// stops waiting.  W: a wavefront's accesses (tree_draft.hpp has those of the GPU).
#pragma once

namespace ot {
namespace {

typedef unsigned long long u64;

// A row's results are in memory once its word is kRowThere.  The workspace needs no preparation: no other value
// counts, and the workgroup that has drafted the tree clears the words of its sequence again, when all of them are there.
// A drafting workgroup does not wait for ever (rows of this launch might not get a place on the chip while other launches'
// drafting workgroups wait there): after `spin` polls it marks the words of all rows that are missing with kRowLate and ends.
// A workgroup that finds that mark as it publishes its row looks whether all rows are there now -- at least the last one sees
// them all -- and then drafts the tree from the beginning.  Should two draft it, both write the same.
constexpr u64 kRowThere = 0x9d3f5be1c7604a2bull, kRowLate = 0x6b1e88d2f0957c43ull;
struct Arrivals {
    u64* there;                   // [rows] of this sequence
    int rows, spin;
    bool wait;                         // false: all rows are there
};

// All rows from `first` on, as seen by one wavefront
template <class W> __device__ __forceinline__ bool rows_there(const W& w, const Arrivals& ar, int first) {
    bool ok = true;
    for (int r0 = first; r0 < ar.rows; r0 += 8 * W::kLanes) { // eight loads per trip to memory
        u64 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = r0 + W::kLanes * u + w.lane;
            x[u] = w.load(ar.there + (r < ar.rows ? r : ar.rows - 1));
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) ok = ok && x[u] == kRowThere;
    }
    return w.all(ok);
}

// One wavefront: marks the rows that are missing, then looks whether all are there after all.  If not, those that are missing
// now were missing before, so all of them are marked, and the last of them to come finds the others there.  (Without the
// second look a row could come, unmarked, between the marks and the visits of rows that found it missing.)
template <class W> __device__ __forceinline__ bool leave_or_all_there(const W& w, const Arrivals& ar) {
    for (int r = w.lane; r < ar.rows; r += W::kLanes) {
        u64 v = w.load(ar.there + r);
        while (v != kRowThere)                                // (a word changes twice at most while this looks at it)
            if (w.swap_if(ar.there + r, v, kRowLate)) break;
    }
    w.stores_done();
    return rows_there(w, ar, 0);
}

// What the wavefronts of a drafting workgroup tell each other (LDS).  A wavefront that stops waiting names the step whose rows it
// has waited for, and behind the next barrier every wavefront looks for that step's number: one that is slow to look may find a
// later number there already, which it must not take for its own.
struct Quit {
    short step;                        // the step whose rows some wavefront has stopped waiting for
    short gone;                        // 1: and rows are missing
};
template <class W> __device__ __forceinline__ void quit_none(const W& w, Quit& q) { w.set(q.step, -1); w.set(q.gone, 0); }
template <class W> __device__ __forceinline__ void quit_waiting(const W& w, Quit& q, int step) { w.set(q.step, step); }
template <class W> __device__ __forceinline__ bool has_quit(const W& w, const Quit& q, int step) { return w.get(q.step) == step; }

// Every wavefront, behind a barrier, some wavefront having quit.  False: another workgroup drafts the tree.
template <class W> __device__ __forceinline__ bool go_alone(const W& w, Quit& q, Arrivals& ar) {
    if (!leave_or_all_there(w, ar)) w.set(q.gone, 1);
    w.barrier();
    ar.wait = false;
    return w.get(q.gone) == 0;
}

// One wavefront, tree drafted from the rows before `first`: clears the words
template <class W> __device__ __forceinline__ void clear_arrivals(const W& w, Arrivals ar, int first) {
    int polls = 0;
    while (ar.wait && !rows_there(w, ar, first)) {
        if (++polls > ar.spin) {
            if (leave_or_all_there(w, ar)) break;
            return;
        }
        w.pause();
    }
    for (int r = w.lane; r < ar.rows; r += W::kLanes) w.store(ar.there + r, 0);
}

// A wavefront of the workgroup that has found its row's word marked: does it draft the tree
template <class W> __device__ __forceinline__ bool take_over(const W& w, const Arrivals& ar) { return rows_there(w, ar, 0); }

}  // namespace
}  // namespace ot
