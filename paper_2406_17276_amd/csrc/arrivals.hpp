// One-shot build as one launch: how the workgroup that drafts a sequence learns which rows are there, and who drafts where it
// stops waiting.  W: a wavefront's accesses (tree_draft.hpp has those of the GPU).
#pragma once

namespace ot {
namespace {

typedef unsigned long long u64;

// A row's results are in memory once its word is kRowThere.  The workspace needs no preparation: no other value
// counts, and the workgroup that has drafted the tree clears the words of its sequence again, when all of them are there.
// A drafting workgroup does not wait for ever (rows of this launch might not get a place on the chip while other launches'
// drafting workgroups wait there): after `spin` polls it marks the words of all rows that are missing with kRowLate, says in the
// sequence's own word that it has done so, and ends.  A workgroup that finds its row's word marked as it publishes the row looks
// whether all rows are there now -- at least the last one sees them all -- and then, once the marks are made, drafts the tree from
// the beginning.  (Sooner, it could clear words that are still being marked, and these marks would be found by the next launch.)
// Should two draft it, both write the same.
constexpr u64 kRowThere = 0x9d3f5be1c7604a2bull, kRowLate = 0x6b1e88d2f0957c43ull, kMarksMade = 0x5c27f4a98e61d03bull;
struct Arrivals {
    u64* there;                        // [rows] of this sequence
    u64* marks;                        // the sequence's own word
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

// One wavefront: marks the rows that are missing.  A look behind it tells who drafts: rows that are missing then were missing
// before, so all of them are marked, and the last of them to come finds the others there.  (A look ahead of it would not do: a row
// could come, unmarked, in between.)
template <class W> __device__ __forceinline__ void mark_missing(const W& w, const Arrivals& ar) {
    for (int r = w.lane; r < ar.rows; r += W::kLanes) {
        u64 v = w.load(ar.there + r);
        while (v != kRowThere)                                // (no word is cleared before kMarksMade: a second try finds the row there)
            if (w.swap_if(ar.there + r, v, kRowLate)) break;
    }
    w.stores_done();
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
    mark_missing(w, ar);
    w.barrier();
    if (w.first) { w.store(ar.marks, kMarksMade); w.stores_done(); }
    if (!rows_there(w, ar, 0)) w.set(q.gone, 1);
    w.barrier();
    ar.wait = false;
    return w.get(q.gone) == 0;
}

// One wavefront, tree drafted from the rows before `first`: clears the words, the sequence's own last (take_over)
template <class W> __device__ __forceinline__ void clear_arrivals(const W& w, Arrivals ar, int first) {
    int polls = 0;
    while (ar.wait && !rows_there(w, ar, first)) {
        if (++polls > ar.spin) {
            mark_missing(w, ar);
            w.store(ar.marks, kMarksMade);
            if (!rows_there(w, ar, 0)) return;
            ar.wait = false;
            break;
        }
        w.pause();
    }
    for (int r = w.lane; r < ar.rows; r += W::kLanes) w.store(ar.there + r, 0);
    if (ar.wait) return;
    w.stores_done();
    if (w.lane == 0) w.store(ar.marks, 0);
}

// A wavefront of a workgroup that has found its row's word marked: does it draft the tree.  The wait ends: whoever marks has a
// place on the chip and says so next, and is seen here or by rows that are cleared, which they are before the sequence's word.
template <class W> __device__ __forceinline__ bool take_over(const W& w, const Arrivals& ar) {
    while (rows_there(w, ar, 0)) {
        if (w.load(ar.marks) == kMarksMade) return true;
        w.pause();
    }
    return false;
}

}  // namespace
}  // namespace ot
