// arrivals.hpp on the host: a drafting workgroup of two wavefronts (a lane each) and a workgroup per row as coroutines that
// change places at every access, in many random orders.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#include "arrivals.hpp"
using namespace ot;

namespace {

struct Task {
    ucontext_t ctx;
    std::vector<char> stack = std::vector<char>(64 * 1024);
    std::function<void()> body;
    int weight;
    bool done, at_barrier;
    int where;
};
ucontext_t g_main;
std::vector<Task*> g_tasks;
Task* g_now;
unsigned long long g_rng;
const char* g_error;
int g_live;                            // wavefronts of the drafting workgroup

unsigned rnd(unsigned n) { g_rng = g_rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(g_rng >> 33) % n; }
void yield() { swapcontext(&g_now->ctx, &g_main); }
void fail(const char* e) { if (!g_error) g_error = e; }
void entry() { g_now->body(); g_now->done = true; yield(); }

// What tree_draft.hpp's wavefront does, with one lane
struct Wave {
    static constexpr int kLanes = 1;
    int lane;
    bool first;
    u64 load(const u64* p) const { yield(); return *p; }
    void store(u64* p, u64 v) const { yield(); *p = v; }
    bool swap_if(u64* p, u64& v, u64 x) const {
        yield();
        if (*p == v) { *p = x; return true; }
        v = *p;
        return false;
    }
    void stores_done() const {}
    bool all(bool ok) const { return ok; }
    void pause() const { g_now->weight = 1 + (int)rnd(8); yield(); }
    void set(short& f, int v) const { yield(); f = (short)v; }
    int get(const short& f) const { yield(); return f; }
    // waits for the other wavefront, which has to be at the same place (or has ended)
    void barrier() const {
        g_now->at_barrier = true;
        while (g_now->at_barrier) {
            int there = 0;
            for (Task* t : g_tasks) there += t->at_barrier;
            if (there < g_live) { yield(); continue; }
            for (Task* t : g_tasks)
                if (t->at_barrier) { t->at_barrier = false; if (t->where != g_now->where) fail("barriers of two places paired"); }
        }
    }
};

struct World {
    std::vector<u64> word;
    std::vector<char> result;          // rows whose results are in memory
    u64 marks;
    Quit quit;
    int drafted;
    std::vector<int> starts;           // rows before step t
};

void use_rows(World& w, int end) {
    for (int r = 0; r < end; ++r)
        if (!w.result[r]) fail("a row is used that is not there");
}

// The waits of draft_tree, with steps that keep all of their candidates: no barrier but the one at a step's end
void drafter(World& world, Arrivals ar, bool first) {
    const Wave w{0, first};
    const int steps = (int)world.starts.size() - 1;
    auto poll = [&](int t) {
        int polls = 0;
        for (;;) {
            bool ok = true;
            for (int r = world.starts[t]; r < world.starts[t + 1]; ++r) ok = w.load(ar.there + r) == kRowThere && ok;
            if (ok) return;
            if (++polls > ar.spin) { quit_waiting(w, world.quit, t); return; }
            w.pause();
        }
    };
    auto on = [&](int t) {
        if (!has_quit(w, world.quit, t)) return true;
        g_now->where = 100 + t;
        return go_alone(w, world.quit, ar);
    };
    if (first) quit_none(w, world.quit);
    g_now->where = 50;
    w.barrier();
    if (ar.wait) poll(0);
    g_now->where = 0;
    w.barrier();
    bool stay = on(0);
    int seen = 0;
    for (int t = 0; stay && t < steps; ++t) {
        seen = world.starts[t + 1];
        if (first) use_rows(world, seen);
        if (t + 1 < steps && ar.wait) poll(t + 1);
        g_now->where = t + 1;
        w.barrier();
        stay = on(t + 1);
        if (stay && t + 2 >= steps && rnd(3) == 0) break;     // (the tree is complete early)
    }
    --g_live;
    if (!stay) return;
    if (first) ++world.drafted;
    else clear_arrivals(w, ar, seen);
}

void row(World& world, Arrivals ar, int r) {
    const Wave w{0, true};
    yield();
    world.result[r] = 1;
    yield();
    const u64 old = world.word[r];
    world.word[r] = kRowThere;
    if (old != kRowLate || !take_over(w, ar)) return;
    use_rows(world, ar.rows);
    ++world.drafted;
    ar.wait = false;
    clear_arrivals(w, ar, ar.rows);
}

}  // namespace

int main(int argc, char** argv) {
    const int runs = argc > 1 ? atoi(argv[1]) : 1000;
    World world;
    world.starts = {0, 1, 2, 4, 5};
    std::vector<Task> tasks(2 + 5);
    for (int run = 0; run < runs; ++run) {
        g_rng = 0x9e3779b97f4a7c15ull * (unsigned)(run + 1);
        world.word.assign(5, rnd(2) ? 0 : 77);
        world.result.assign(5, 0);
        world.marks = rnd(2) ? 0 : 77;
        world.quit = Quit{9, 9};
        world.drafted = 0;
        g_live = 2;
        g_error = nullptr;
        Arrivals ar{};
        ar.there = world.word.data(); ar.rows = 5; ar.spin = (int)rnd(4); ar.wait = true;
        ar.marks = &world.marks;
        g_tasks.clear();
        for (int i = 0; i < 7; ++i) {
            Task& t = tasks[i];
            if (i < 2) t.body = [&world, ar, i] { drafter(world, ar, i == 0); };
            else t.body = [&world, ar, i] { row(world, ar, i - 2); };
            t.weight = 1 << rnd(10);                          // some orders are fair, in others one stands still for long
            t.done = t.at_barrier = false;
            t.where = -1;
            getcontext(&t.ctx);
            t.ctx.uc_stack.ss_sp = t.stack.data();
            t.ctx.uc_stack.ss_size = t.stack.size();
            t.ctx.uc_link = nullptr;
            makecontext(&t.ctx, entry, 0);
            g_tasks.push_back(&t);
        }
        for (int moves = 0; !g_error; ++moves) {
            if (rnd(16) == 0) g_tasks[rnd(7)]->weight = 1 << rnd(10);
            int total = 0;
            for (Task* t : g_tasks) total += t->done || (t->at_barrier && g_live > 1) ? 0 : t->weight;
            bool all_done = true;
            for (Task* t : g_tasks) all_done = all_done && t->done;
            if (all_done) break;
            if (!total) { fail("a wait without end"); break; }
            if (moves > 200000) { fail("too many moves"); break; }
            int at = (int)rnd(total);
            for (Task* t : g_tasks) {
                if (t->done || (t->at_barrier && g_live > 1)) continue;
                at -= t->weight;
                if (at < 0) { g_now = t; break; }
            }
            swapcontext(&g_main, &g_now->ctx);
        }
        if (!g_error && !world.drafted) fail("nobody has drafted the tree");
        for (u64 v : world.word)
            if (!g_error && (v == kRowThere || v == kRowLate)) fail("a word is left set");
        if (!g_error && world.marks != 0 && world.marks != 77) fail("the sequence's word is left set");
        if (g_error) { printf("run %d: %s\n", run, g_error); return 1; }
    }
    printf("ok %d\n", runs);
    return 0;
}
