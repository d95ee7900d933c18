// CPU model of the step kernel's cross-workgroup protocols, run under
// ThreadSanitizer: one host thread per workgroup, std::atomic in place of the
// device-coherent atomics, and the protocol arithmetic of the library itself
// (kl_sync.h, compiled here for the host).
//
// The device code orders its data before a signal by completing its stores
// (s_waitcnt vmcnt(0)) before the relaxed arrival atomic is issued, and a
// waiter issues its data loads only after its poll has seen the count; in the
// C++ memory model that is a release on the arrival and an acquire on the
// poll, which is what the model uses.  Tagged words need no ordering at all:
// value and tag travel in one atomic 8-byte access (relaxed here).
//
// Checks, each over several launches in a row (counters never reset):
//   1. grid barrier: no thread passes barrier k before every thread has
//      written its slot for k; launches recover their epoch from their own
//      group's counter (uneven group sizes: 20 threads on 16 counters);
//   2. watchdog: a launch in which one thread never arrives ends in every
//      thread with the error flag set, instead of hanging;
//   3. tagged hand-offs: readers accept exactly the current layer's values,
//      never an earlier layer's or step's, across the tag wrap;
//   4. a missing tagged writer trips the watchdog too;
//   5. RMSNorm slices: a product that waits for staged_slices of a chunk reads
//      no column whose slice is not complete, for K ranges that start and end
//      anywhere in a slice;
//   6. the epoch: in a launch of the step's last phase alone, a workgroup that
//      starts after others are done still finds the step's own tags;
//   7. the token loop's argmax keys: a step's maximum is its own;
//   8. reuse of the per-sequence path's word buffers: eight buffers written
//      again in every layer without any barrier, each phase reading and writing
//      what the kernel's does (workgroups without rows in a phase read
//      nothing in it): no word is overwritten before its last reader has it.
// Prints "sync model OK" and exits 0, else prints the failure and exits 1.
// With --plant-early-barrier it runs check 1 with a planted off-by-one barrier
// target, with --plant-one-slice check 5 with a chunk that waits for the slice
// of its first column alone, with --plant-early-epoch check 6 with the epoch
// advanced by workgroup 0 when it is done, with --plant-own-keys check 7 with
// each step clearing its own set of keys, with --plant-idle-reader check 8 with
// a workgroup that reads a layer's input without having rows of its product,
// which the check (or ThreadSanitizer) must report.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <thread>
#include <vector>

#include "kl_sync.h"

using namespace kl;

namespace {

// polls before a wait gives up (the device allows 2^22 polls of about a
// microsecond each; here every poll past the first 64 yields the CPU)
constexpr int kSpin = 1 << 18;

int g_fail = 0;
int g_plant = 0;   // a planted mistake; 1: barrier k waits for barrier k - 1's target
int g_plant_slice = 0;   // 1: a chunk waits for one slice
int g_plant_keys = 0;    // 1: a step clears the keys it takes its own maximum into
int g_plant_idle = 0;    // 1: a workgroup without rows reads the residual
int g_plant_epoch = 0;   // 1: workgroup 0 advances the epoch when it is done
void check(bool ok, const char *what) {
    if (!ok) {
        std::fprintf(stderr, "FAIL: %s\n", what);
        g_fail = 1;
    }
}

struct Grid {
    int nwg, ng;
    std::vector<std::atomic<unsigned long long>> cnt;   // one per group
    std::atomic<int> err{0};
    explicit Grid(int n) : nwg(n), ng(bar_group_count(n)), cnt(bar_group_count(n)) {
        for (auto &c : cnt) c.store(0);
    }
};

// One workgroup's view of a launch: bases recovered from its own group.
struct Launch {
    Grid &G;
    int w;
    std::vector<unsigned long long> base;
    Launch(Grid &g, int w_) : G(g), w(w_), base(g.ng) {
        const int own = w % G.ng;
        const unsigned long long c = G.cnt[own].load(std::memory_order_acquire);
        for (int g = 0; g < G.ng; ++g) base[g] = bar_launch_base(c, G.nwg, G.ng, own, g);
    }
    void arrive() { G.cnt[w % G.ng].fetch_add(1, std::memory_order_release); }
    // false when the wait gave up (the error flag is then set)
    bool wait(int k) {
        for (int spins = 1;; ++spins) {
            bool done = true;
            for (int g = 0; g < G.ng; ++g)
                done = done && bar_reached(G.cnt[g].load(std::memory_order_acquire),
                                           bar_target(base[g], k - g_plant, G.nwg, G.ng, g));
            if (done) return true;
            if ((spins & 63) == 0 && G.err.load(std::memory_order_relaxed)) return false;
            if (spins >= kSpin) {
                G.err.store(1, std::memory_order_relaxed);
                return false;
            }
            if (spins > 64) std::this_thread::yield();
        }
    }
};

template <class F>
void run_threads(int n, F &&f) {
    std::vector<std::thread> t;
    for (int w = 0; w < n; ++w) t.emplace_back(f, w);
    for (auto &x : t) x.join();
}

// 1. barriers over several launches; plain (non-atomic) data, ordered by the
// barrier alone: TSan reports a race if the protocol lets a reader through early
void test_barrier(int nwg, int launches, int nbar) {
    Grid G(nwg);
    std::vector<int> slot(nwg * nbar, -1);
    for (int L = 0; L < launches; ++L) {
        run_threads(nwg, [&](int w) {
            Launch me(G, w);
            for (int k = 0; k < nbar; ++k) {
                slot[k * nwg + w] = L * 1000 + k;
                me.arrive();
                if (!me.wait(k)) return;
                for (int v = 0; v < nwg; ++v)
                    if (slot[k * nwg + v] != L * 1000 + k) G.err.store(2);
            }
        });
        check(G.err.load() == 0, "barrier: a thread passed before every slot was written");
    }
    for (int g = 0; g < G.ng; ++g)
        check(G.cnt[g].load() ==
                  (unsigned long long)launches * nbar * bar_group_size(nwg, G.ng, g),
              "barrier: counters end at launches x barriers x group size");
}

// 2. a missing arrival ends the launch through the watchdog
void test_watchdog(int nwg) {
    Grid G(nwg);
    run_threads(nwg, [&](int w) {   // a clean launch first (2 barriers)
        Launch me(G, w);
        for (int k = 0; k < 2; ++k) {
            me.arrive();
            me.wait(k);
        }
    });
    check(G.err.load() == 0, "watchdog: clean launch");
    std::atomic<int> returned{0};
    run_threads(nwg, [&](int w) {
        Launch me(G, w);
        me.arrive();
        me.wait(0);
        if (w != 3) me.arrive();   // workgroup 3 never arrives on barrier 1
        me.wait(1);
        returned.fetch_add(1);
    });
    check(G.err.load() == 1, "watchdog: a missing arrival sets the error flag");
    check(returned.load() == nwg, "watchdog: every thread returned");
}

// 3. tagged hand-offs: per step and layer, writers publish words, readers
// (after the barrier that separates uses of the buffer, as in the kernel) poll
// until current and check the value
void test_tagged(int nwg, int steps, int layers, unsigned first_epoch) {
    Grid G(nwg);
    const int nwords = 3 * nwg;
    std::vector<std::atomic<unsigned long long>> buf(nwords);
    for (auto &x : buf) x.store(0);   // cleared memory: tag 0, never current
    unsigned epoch = first_epoch;
    for (int s = 0; s < steps; ++s) {
        const unsigned e = epoch;
        check(e != 0 && e + (unsigned)layers - 1u >= e, "tags: a step's range holds no 0, no wrap");
        run_threads(nwg, [&](int w) {
            Launch me(G, w);
            for (int l = 0; l < layers; ++l) {
                const unsigned tag = e + (unsigned)l;
                for (int i = w; i < nwords; i += nwg)   // write my words of layer l
                    buf[i].store(ll_word((unsigned)(s * 7919 + l * 131 + i), tag),
                                 std::memory_order_relaxed);
                // read every word of layer l (written by others)
                for (int i = 0; i < nwords; ++i) {
                    unsigned long long v = 0;
                    for (int spins = 1;; ++spins) {
                        v = buf[i].load(std::memory_order_relaxed);
                        if (ll_current(v, tag)) break;
                        if (spins >= kSpin || G.err.load(std::memory_order_relaxed)) {
                            G.err.store(1);
                            return;
                        }
                        if (spins > 64) std::this_thread::yield();
                    }
                    if (ll_value(v) != (unsigned)(s * 7919 + l * 131 + i)) G.err.store(3);
                }
                // (here a grid barrier separates the buffer's uses; without: 8)
                me.arrive();
                if (!me.wait(l)) return;
            }
        });
        check(G.err.load() == 0, "tags: every value read is the current layer's");
        const unsigned next = ll_next_epoch(e, layers);
        check(next == 1u || next == e + (unsigned)layers, "tags: the next range follows or restarts");
        check(next + (unsigned)layers - 1u >= next, "tags: the next range does not wrap");
        epoch = next;
    }
}

// 4. a word that is never written trips the watchdog
void test_tagged_missing_writer() {
    std::atomic<unsigned long long> word{ll_word(5, 41)};   // last step's tag
    std::atomic<int> err{0};
    std::thread t([&] {
        for (int spins = 1;; ++spins) {
            if (ll_current(word.load(std::memory_order_relaxed), 42)) return;
            if (spins >= kSpin) {
                err.store(1);
                return;
            }
        }
    });
    t.join();
    check(err.load() == 1, "tags: a stale word is never taken as current");
}

// 5. every column of every chunk of every K range (KT k-tiles in KS equal
// slices, as the host may choose them) lies in a slice that the chunk waits
// for, and no other slice is waited for
SliceRange waited_slices(int col0, int width, int c, int chunk) {
    SliceRange r = staged_slices(col0, width, c, chunk);
    if (g_plant_slice) r.end = r.first + 1;
    return r;
}
void test_slice_cover(int chunk) {
    const int tile = 64;
    bool covered = true, tight = true;
    for (int KT = 1; KT <= 320; ++KT)
        for (int KS = 1; KS <= 16; ++KS) {
            if (KT % KS) continue;
            const int width = KT / KS * tile;
            for (int ks = 0; ks < KS; ++ks) {
                const int col0 = ks * width;
                for (int c = 0; c * chunk < width; ++c) {
                    const SliceRange r = waited_slices(col0, width, c, chunk);
                    std::vector<int> touched;
                    for (int k = c * chunk; k < width && k < (c + 1) * chunk; ++k) {
                        const int sl = (col0 + k) / chunk;
                        covered = covered && sl >= r.first && sl < r.end;
                        if (touched.empty() || touched.back() != sl) touched.push_back(sl);
                    }
                    tight = tight && r.end - r.first == (int)touched.size();
                }
            }
        }
    check(covered, "slices: a chunk's columns lie in the slices it waits for");
    check(g_plant_slice || tight, "slices: a chunk waits for no other slice");
}
// the same with threads: the row is plain data, ordered by the slice counters
// alone; the last slice comes late
void test_slice_handoff(int KT, int KS, int chunk) {
    const int tile = 64, H = KT * tile, ns = (H + chunk - 1) / chunk, width = KT / KS * tile;
    std::vector<int> row(H, -1);
    std::vector<std::atomic<unsigned>> cnt(ns);
    for (auto &c : cnt) c.store(0);
    std::atomic<int> bad{0};
    run_threads(ns + KS, [&](int w) {
        if (w < ns) {   // the producer of slice w
            for (int y = 0; y < 200 * w; ++y) std::this_thread::yield();
            for (int i = w * chunk; i < H && i < (w + 1) * chunk; ++i) row[i] = i;
            cnt[w].fetch_add(1, std::memory_order_release);
            return;
        }
        const int col0 = (w - ns) * width;
        for (int c = 0; c * chunk < width; ++c) {
            const SliceRange r = waited_slices(col0, width, c, chunk);
            for (int s = r.first; s < r.end; ++s)
                for (int spins = 0; cnt[s].load(std::memory_order_acquire) == 0; ++spins) {
                    if (spins >= kSpin) { bad.store(1); return; }
                    std::this_thread::yield();
                }
            for (int k = c * chunk; k < width && k < (c + 1) * chunk; ++k)
                if (row[col0 + k] != col0 + k) bad.store(1);
        }
    });
    check(bad.load() == 0, "slices: every column staged is complete");
}

// 6. the step's last phase as a launch of its own: each workgroup reads the
// epoch when it starts, polls for words of the layers' launches, is done;
// workgroup 'late' starts once workgroup 0 is done (and every other one is, in
// every second step)
void test_epoch(int nwg, int steps, int layers, int late) {
    std::atomic<unsigned> epoch{1}, arrivals{0};
    std::vector<std::atomic<unsigned long long>> x(nwg);   // the last residual
    std::atomic<int> err{0};
    for (int s = 0; s < steps; ++s) {
        const unsigned e = epoch.load();
        for (int i = 0; i < nwg; ++i)
            x[i].store(ll_word((unsigned)(s * 17 + i), e + (unsigned)layers));
        std::atomic<int> done0{0}, done{0};
        run_threads(nwg, [&](int w) {
            if (w == late)
                while (done0.load() == 0 || (s % 2 && done.load() < nwg - 1)) std::this_thread::yield();
            const unsigned mine = epoch.load(std::memory_order_relaxed);
            for (int i = 0; i < nwg; ++i)
                for (int spins = 1;; ++spins) {
                    const unsigned long long v = x[i].load(std::memory_order_relaxed);
                    if (ll_current(v, mine + (unsigned)layers)) {
                        if (ll_value(v) != (unsigned)(s * 17 + i)) err.store(3);
                        break;
                    }
                    if (spins >= kSpin || err.load()) {
                        err.store(1);
                        break;
                    }
                }
            const bool last = epoch_last_arrival(arrivals.fetch_add(1), nwg);
            if (last) arrivals.store(0);
            if (g_plant_epoch ? w == 0 : last) epoch.store(ll_next_epoch(mine, layers + 1));
            if (w == 0) done0.store(1);
            done.fetch_add(1);
        });
        check(err.load() == 0, "epoch: a late workgroup finds the step's own tags");
        check(epoch.load() == ll_next_epoch(e, layers + 1) && arrivals.load() == 0,
              "epoch: advanced once, the counter cleared");
    }
}

// 7. a token loop: step n's workgroups take the maximum of their keys, workgroup
// 0 clears a set when the others are done; loops of different lengths in a row
void test_keys(int nwg, const std::vector<int> &loops) {
    std::vector<std::atomic<unsigned long long>> keys(kKeySlots);
    for (auto &k : keys) k.store(0);
    std::atomic<int> bad{0};
    for (int steps : loops) {
        unsigned long long want = 0;
        for (int n = 0; n < steps; ++n) {
            std::atomic<int> done{1};
            // (every step's largest key is below the ones of the steps before)
            const unsigned long long top = 100000ull - 100ull * (unsigned)n;
            run_threads(nwg, [&](int w) {
                if (w == 0) {
                    while (done.load() < nwg) std::this_thread::yield();
                    keys[key_slot(g_plant_keys ? n : n + 1)].store(0);
                    return;
                }
                if (n > 0 && keys[key_slot(n - 1)].load() != want) bad.store(1);
                const unsigned long long k = top + (unsigned)w;
                unsigned long long o = keys[key_slot(n)].load();
                while (o < k && !keys[key_slot(n)].compare_exchange_weak(o, k)) {}
                done.fetch_add(1);
            });
            want = top + (unsigned)(nwg - 1);
        }
        check(keys[key_slot(steps - 1)].load() == want, "keys: a step's maximum is its own");
        keys[key_slot(0)].store(0);   // the loop's last launch
    }
    check(bad.load() == 0, "keys: every workgroup reads the step before's maximum");
}

// 8. one step of the per-sequence path at a time: nwg workgroups, of which the
// last has no rows in the layers; B sequences, each in its turn inside a phase
// (a pass that they share reads and writes the same words at once)
struct Words {
    std::vector<std::atomic<unsigned long long>> w;
    explicit Words(int n) : w(n) { for (auto &x : w) x.store(0); }
};
void test_reuse(int B, int steps, int layers, unsigned seed) {
    // owners of the residual rows: workgroups 0 .. 2, two rows each; q/k/v and
    // attention: 2 heads of 3 workgroups, the third without units; merge: one
    // output per workgroup 0 .. 3; FFN: 2 column blocks of 3 workgroups, the
    // first of a block without gate/up rows, the last without down rows
    constexpr int kWg = 8, H = 6, Q = 4, P = 2, O = 4, M = 2, J = 2;
    Words xb(B * H), xa(B * H), q(B * 2 * Q), po(B * 2 * P * 2), o(B * O), m(B * J * M), dp(B * J * H);
    std::atomic<unsigned> epoch{1}, arrivals{0};
    std::atomic<int> err{0};
    for (int s = 0; s < steps; ++s) {
        const unsigned e = epoch.load();
        run_threads(kWg, [&](int w) {
            unsigned rng = seed + 977u * (unsigned)w + 131071u * (unsigned)s;
            const unsigned mine = epoch.load(std::memory_order_relaxed);
            auto value = [&](int id, int i, int l) { return (unsigned)(s * 1000003 + l * 1009 + id * 97 + i); };
            auto pause = [&]() {   // (now and then a workgroup falls far behind)
                rng = rng * 1664525u + 1013904223u;
                const int n = (rng >> 20) % 16 == 0 ? 300 : (rng >> 24) % 4;
                for (int k = 0; k < n; ++k) std::this_thread::yield();
            };
            auto put = [&](Words &b, int id, int i, int l) {
                b.w[i].store(ll_word(value(id, i, l), mine + (unsigned)l), std::memory_order_relaxed);
            };
            auto get = [&](Words &b, int id, int i, int l) {
                for (int spins = 1;; ++spins) {
                    const unsigned long long v = b.w[i].load(std::memory_order_relaxed);
                    if (ll_current(v, mine + (unsigned)l)) {
                        if (ll_value(v) != value(id, i, l)) err.store(3);
                        return;
                    }
                    // (a newer tag: overwritten before this reader had it)
                    if ((unsigned)(v >> 32) > mine + (unsigned)l || spins >= kSpin) err.store(4);
                    if (err.load(std::memory_order_relaxed)) return;
                    std::this_thread::yield();
                }
            };
            const bool owner = w < 3, layer = w < 6;
            const int g = w / 3, part = w % 3;
            if (owner)
                for (int i = 0; i < 2 * B; ++i) put(xb, 0, (i / 2) * H + 2 * w + i % 2, 0);
            for (int l = 0; l < layers; ++l) {
                pause();
                if (layer || (g_plant_idle && w == kWg - 1))   // q/k/v
                    for (int b = 0; b < B; ++b) {
                        for (int i = 0; i < H; ++i) get(xb, 0, b * H + i, l);
                        if (!layer) continue;
                        for (int i = part; i < Q; i += 3) put(q, 1, (b * 2 + g) * Q + i, l);
                    }
                pause();
                if (layer && part < P)                         // attention shares
                    for (int b = 0; b < B; ++b) {
                        for (int i = 0; i < Q; ++i) get(q, 1, (b * 2 + g) * Q + i, l);
                        for (int i = 0; i < 2; ++i) put(po, 2, ((b * 2 + g) * P + part) * 2 + i, l);
                    }
                pause();
                if (w < O)                                     // merge
                    for (int b = 0; b < B; ++b) {
                        for (int i = 0; i < 2 * P; ++i) get(po, 2, (b * 2 + w / 2) * P * 2 + i, l);
                        put(o, 3, b * O + w, l);
                    }
                if (owner)                                     // O projection
                    for (int b = 0; b < B; ++b) {
                        for (int i = 0; i < O; ++i) get(o, 3, b * O + i, l);
                        for (int i = 0; i < 2; ++i) put(xa, 4, b * H + 2 * w + i, l);
                    }
                pause();
                if (layer && part > 0)                         // gate/up
                    for (int b = 0; b < B; ++b) {
                        for (int i = 0; i < H; ++i) get(xa, 4, b * H + i, l);
                        put(m, 5, (b * J + g) * M + part - 1, l);
                    }
                pause();
                if (layer && part < 2)                         // down
                    for (int b = 0; b < B; ++b) {
                        for (int i = 0; i < M; ++i) get(m, 5, (b * J + g) * M + i, l);
                        for (int i = 3 * part; i < 3 * part + 3; ++i) put(dp, 6, (b * J + g) * H + i, l);
                    }
                if (owner) {                                   // the owners' sums
                    for (int b = 0; b < B; ++b)
                        for (int j = 0; j < J; ++j)
                            for (int i = 0; i < 2; ++i) get(dp, 6, (b * J + j) * H + 2 * w + i, l);
                    for (int i = 0; i < 2 * B; ++i) put(xb, 0, (i / 2) * H + 2 * w + i % 2, l + 1);
                }
            }
            pause();
            if (w % 2)                                         // head
                for (int i = 0; i < B * H; ++i) get(xb, 0, i, layers);
            if (epoch_last_arrival(arrivals.fetch_add(1), kWg)) {
                arrivals.store(0);
                epoch.store(ll_next_epoch(mine, layers + 1));
            }
        });
        check(err.load() == 0, "reuse: every word is read before it is overwritten");
        check(epoch.load() == ll_next_epoch(e, layers + 1), "reuse: the epoch is advanced once");
        if (err.load()) return;
    }
}

}  // namespace

int main(int argc, char **argv) {
    if (argc > 1 && std::string(argv[1]) == "--plant-early-barrier") {
        // the model must catch a barrier that lets threads through one early
        g_plant = 1;
        test_barrier(20, 2, 5);
        return g_fail ? 1 : 0;
    }
    if (argc > 1 && std::string(argv[1]) == "--plant-one-slice") {
        g_plant_slice = 1;
        test_slice_cover(512);
        test_slice_handoff(12, 2, 512);
        return g_fail ? 1 : 0;
    }
    if (argc > 1 && std::string(argv[1]) == "--plant-early-epoch") {
        g_plant_epoch = 1;
        test_epoch(8, 2, 3, 5);
        return g_fail ? 1 : 0;
    }
    if (argc > 1 && std::string(argv[1]) == "--plant-own-keys") {
        g_plant_keys = 1;
        test_keys(6, {2});
        return g_fail ? 1 : 0;
    }
    if (argc > 1 && std::string(argv[1]) == "--plant-idle-reader") {
        g_plant_idle = 1;
        for (unsigned seed = 1; seed <= 40 && !g_fail; ++seed) test_reuse(1, 4, 6, seed);
        return g_fail ? 1 : 0;
    }
    // group sizes: 20 threads on 16 counters (sizes 2 and 1); 5 on 5
    test_barrier(20, 4, 5);
    test_barrier(5, 3, 7);
    test_watchdog(20);
    test_tagged(12, 4, 3, 1u);
    // near the top of the tag space: the range restarts at 1 instead of wrapping
    test_tagged(12, 4, 3, 0xFFFFFFFFu - 8u);
    test_tagged_missing_writer();
    test_slice_cover(512);
    test_slice_handoff(12, 2, 512);    // 768 columns in 2 K slices of 384
    test_slice_handoff(40, 8, 512);    // 2560 in 8 of 320
    test_slice_handoff(80, 4, 512);    // 5120 in 4 of 1280 (three chunks each)
    test_epoch(8, 6, 3, 5);
    test_epoch(1, 3, 3, 1);
    test_keys(6, {1, 5, 2, 3, 4, 1, 1});
    for (unsigned seed = 1; seed <= 12; ++seed) {
        test_reuse(1, 4, 6, seed);
        test_reuse(3, 3, 5, seed + 100);
    }
    // the epoch arithmetic on its own
    check(ll_next_epoch(0, 32) == 1, "epoch: 0 restarts at 1");
    check(ll_next_epoch(1, 32) == 33, "epoch: consecutive ranges");
    check(ll_next_epoch(0xFFFFFFFFu - 63u, 32) == 1, "epoch: restart before the top");
    check(bar_launch_base(7, 20, 16, 3, 0) == 6 && bar_launch_base(7, 20, 16, 3, 5) == 3,
          "barrier: base from the own group's count (sizes 2 and 1)");
    if (g_fail) return 1;
    std::printf("sync model OK\n");
    return 0;
}
