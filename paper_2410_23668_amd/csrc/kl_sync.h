// Arithmetic of the step kernel's cross-workgroup protocols, shared by the
// device code and by the CPU model of the protocols in the tests (compiled
// there with KL_HD defined empty).  Nothing here touches memory.
//
// Grid barrier.  nwg workgroups arrive on ng = min(kBarGroups, nwg) monotonic
// 64-bit counters, workgroup w on counter w % ng, which therefore counts
// group_size(g) arrivals per barrier.  The counters are never reset: after E
// complete barriers counter g holds E * group_size(g).  At launch start a
// workgroup reads its own group's counter c and recovers E = c / size (its
// own group cannot have completed barrier E before it arrives, so c is below
// (E + 1) size); barrier k of the launch is then complete when every counter
// g has reached (E + k + 1) group_size(g).
//
// Tagged hand-offs.  A value crossing workgroups travels in one 8-byte word
// with the tag of the step and layer that wrote it (value in the low 32
// bits, tag in the high 32 bits); a reader accepts a word whose tag is the
// current one.  Step s uses tags epoch_s .. epoch_s + L (layer l's words and its
// input residual; the head's input): L + 1 of them;
// the next step's range starts right after, and restarts at 1 before it
// would reach 2^32, so no step's range contains 0, the tag of cleared memory.
// The epoch lives in device memory.  Every workgroup of a launch reads it when
// it starts, and the step's last phase advances it, where workgroups that start
// late may still have to read it (nothing else of that launch orders them).  So
// each workgroup adds one to an arrival counter after its own read, and the
// last to arrive stores the next epoch and clears the counter.
//
// Argmax keys of the token loop: three sets in turn.  Step n's head takes the
// maximum into set key_slot(n) while the step still reads its tokens from
// set key_slot(n - 1), and clears set key_slot(n + 1), which nothing else
// touches in that step: the clearing is ordered before its use by the launch
// boundary alone, whatever the order of the workgroups within a launch.
//
// RMSNorm slices (matrix-core path).  A normalised row is handed over in slices
// of 'chunk' columns, each with a counter; a product stages its K range in
// chunks of as many columns, counted from the range's own first column, which
// need not be a multiple of them: a chunk may lie in two slices, and waits for
// both.
#pragma once

#include <stdint.h>

#ifndef KL_HD
#define KL_HD __host__ __device__
#endif

namespace kl {

constexpr int kSyncBarGroups = 16;   // first level of the grid barrier

KL_HD inline int bar_group_count(int nwg) { return nwg < kSyncBarGroups ? nwg : kSyncBarGroups; }

// Arrivals per barrier on counter g (workgroups w with w % ng == g).
KL_HD inline unsigned bar_group_size(int nwg, int ng, int g) {
    return (unsigned)(nwg / ng + (g < nwg % ng ? 1 : 0));
}

// The value counter g starts this launch at, from the own group's counter c
// (own group og).
KL_HD inline unsigned long long bar_launch_base(unsigned long long own_count, int nwg, int ng,
                                               int og, int g) {
    const unsigned long long epoch = own_count / bar_group_size(nwg, ng, og);
    return epoch * bar_group_size(nwg, ng, g);
}

// Counter g's value once barrier k of the launch is complete.
KL_HD inline unsigned long long bar_target(unsigned long long base, int k, int nwg, int ng,
                                          int g) {
    return base + (unsigned long long)(k + 1) * bar_group_size(nwg, ng, g);
}

// Wrap-safe "counter has reached target" for monotonic 64-bit counters.
KL_HD inline bool bar_reached(unsigned long long count, unsigned long long target) {
    return (long long)(count - target) >= 0;
}

KL_HD inline unsigned long long ll_word(unsigned value, unsigned tag) {
    return ((unsigned long long)tag << 32) | value;
}
KL_HD inline bool ll_current(unsigned long long word, unsigned tag) {
    return (unsigned)(word >> 32) == tag;
}
KL_HD inline unsigned ll_value(unsigned long long word) { return (unsigned)word; }

// The first tag of the step after one whose range started at 'prev', for a
// step of n_layers tags (0 < n_layers < 2^30).
KL_HD inline unsigned ll_next_epoch(unsigned prev, int n_layers) {
    const unsigned L = (unsigned)n_layers;
    if (prev == 0 || prev > 0xFFFFFFFFu - 2u * L) return 1u;   // restart before wrapping
    return prev + L;
}

// Whether the workgroup that found 'before' arrivals is the launch's last one.
KL_HD inline bool epoch_last_arrival(unsigned before, int nwg) {
    return before == (unsigned)nwg - 1u;
}

// The set of argmax keys of step n of a token loop (n >= -1).
constexpr int kKeySlots = 3;
KL_HD inline int key_slot(int n) { return (n + kKeySlots) % kKeySlots; }

// The slices that hold columns of chunk c of the K range [col0, col0 + width).
struct SliceRange { int first, end; };
KL_HD inline SliceRange staged_slices(int col0, int width, int c, int chunk) {
    const int k0 = col0 + c * chunk;
    const int k1 = k0 + chunk < col0 + width ? k0 + chunk : col0 + width;
    return SliceRange{k0 / chunk, (k1 - 1) / chunk + 1};
}

}  // namespace kl
