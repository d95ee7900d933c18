// Arithmetic of the shares that workgroups take of a phase's work, shared by
// the device code and by the CPU test of the shares (compiled there with KL_HD
// defined empty).
#pragma once

#ifndef KL_HD
#define KL_HD __host__ __device__
#endif

namespace kl {

// Attention, per-sequence path.  The T units of a batch of B sequences are
// dealt to the Sg workgroups of a KV head in equal shares, which may cross from
// one sequence into the next.  A share's second segment costs 6 to 8 us, as
// much as kSegCost units (8 KiB each, 0.33 us at a workgroup's part of the
// bandwidth).  So where shares are short (below kSegUnits units) they keep to
// one sequence each, unless the largest share would then be more than kSegCost
// units above the equal one: with few workgroups per KV head and one long
// context among short ones it may be several times that.  Batch 4, 32 KV heads
// of 128 (8 workgroups each), 4 layers, by sequence and equal: contexts 8000
// and 3 x 500 (largest share 126 units against 75) 741 and 706 us; 1500 and
// 3 x 32 (24 against 13) 630 and 640.
// Sequence b's workgroups are one, and of the Sg - B others the part that its
// units have of the batch's.
constexpr int kSegUnits = 96;
constexpr int kSegCost = 20;
struct SeqParts { int first, span, count; };   // workgroups of a sequence; those with units
KL_HD inline SeqParts seq_parts(int Sg, int B, int b, int before, int units, int T) {
    const int rest = Sg - B;
    const int p0 = b + (int)((long long)rest * before / T);
    const int p1 = b + 1 + (int)((long long)rest * (before + units) / T);
    const int span = p1 - p0;
    return SeqParts{p0, span, span < units ? span : units};
}
// (one sequence: the same either way)
KL_HD inline bool seg_short(int Sg, int B, int T) { return B <= Sg && T < kSegUnits * Sg; }
KL_HD inline bool seg_by_sequence(int Sg, int T, int most) {
    return most <= (T + Sg - 1) / Sg + kSegCost;
}

}  // namespace kl
