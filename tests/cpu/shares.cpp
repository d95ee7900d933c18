// The shares that workgroups take of a phase's work (kl_shares.h).
// Attention of the per-sequence path: shares that keep to a sequence each cover
// every sequence's units once, and they are taken only where the largest one is
// within kSegCost units of an equal share.
// Prints "shares OK" and exits 0, else prints the failures and exits 1.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "kl_shares.h"

using namespace kl;

namespace {

int g_fail = 0;
void check(bool ok, const char *what, int a, int b) {
    if (ok || ++g_fail > 20) return;
    std::fprintf(stderr, "FAIL: %s (%d, %d)\n", what, a, b);
}

// the largest share by sequence, and whether such shares are taken
bool by_sequence(int Sg, const std::vector<int> &units, int &most) {
    const int B = (int)units.size();
    int T = 0, before = 0, next = 0;
    for (int u : units) T += u;
    most = 0;
    if (!seg_short(Sg, B, T)) return false;
    for (int b = 0; b < B; before += units[b++]) {
        const SeqParts q = seq_parts(Sg, B, b, before, units[b], T);
        check(q.first == next && q.span >= 1, "a sequence's workgroups follow the last one's", Sg, b);
        check(q.count >= 1 && q.count <= q.span && q.count <= units[b], "workgroups with units", Sg, b);
        next = q.first + q.span;
        most = std::max(most, (units[b] + q.count - 1) / q.count);
    }
    check(next == Sg, "every workgroup has a sequence", Sg, B);
    return seg_by_sequence(Sg, T, most);
}

void attention() {
    int most;
    // one long context among short ones, few workgroups per KV head
    check(!by_sequence(8, {501, 32, 32, 32}, most) && most == 126, "8 workgroups", most, 75);
    check(!by_sequence(4, {370, 2, 2, 2}, most) && most == 370, "4 workgroups", most, 94);
    // the 8B shape's ragged prompts, 32 workgroups per KV head
    check(by_sequence(32, {94, 79, 63}, most), "32 workgroups", most, 8);
    check(by_sequence(32, {1, 1, 1, 1}, most) && most == 1, "empty contexts", most, 1);
    std::srand(7);
    for (int i = 0; i < 200000; ++i) {
        const int Sg = 1 + std::rand() % 256, B = 1 + std::rand() % 7;
        std::vector<int> units(B);
        int T = 0;
        for (int &u : units) T += u = 1 + std::rand() % (1 << (std::rand() % 14));
        if (by_sequence(Sg, units, most))
            check(most <= (T + Sg - 1) / Sg + kSegCost, "the largest share", most, Sg);
    }
}

}  // namespace

int main() {
    attention();
    if (g_fail) return 1;
    std::printf("shares OK\n");
    return 0;
}
