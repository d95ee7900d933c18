// The step kernel's work geometry and the layout of its dynamic LDS for a
// model.  Shared by the host runtime and by the CPU test of the layout
// (compiled there with KL_HD defined empty).
#pragma once

#include <algorithm>

#include "kl_layout.h"
#include "kl_sync.h"

namespace kl {

// Work geometry shared by host and device.
constexpr int kWaves = 8;                 // compute waves per workgroup
constexpr int kCtlWave = kWaves;          // the control wave: barriers and counters only
constexpr int kThreads = (kWaves + 1) * 64;   // threads per workgroup
constexpr int kRgBatch = 16;              // row groups reduced per LDS round
// Batched steps (the matrix-core path) run the weight products on the matrix
// cores.  An activation x enters them as two bf16 terms, hi = bf16(x) and
// lo = bf16(x - hi), both multiplied into the same fp32 accumulators (about
// 16 significant bits of x instead of 8).  Activations are staged in LDS in
// chunks of kGemmChunkK columns for up to kGemmBatch sequences at a time,
// weight rows in blocks of 16.
constexpr int kMfmaBatch = 8;
// Up to kMultiSeq sequences share one pass of the GEMV engine: each weight
// tile is applied to every staged vector, so the weights stream once.  8
// layers of the 8B shape, 4096 cached positions, batch 4: 1162 us with the
// pass on the matrix cores, 1195 on the vector units.  Against the matrix-core
// engine the vector-unit pass took 4.35 ms to 5.0 for all 32 layers, both
// before the residual rows had owners.  Dense models take that engine from
// the batch on that does not share a pass: kMultiSeq + 1, 3 with many heads
// (lds_layout_for), or kBatchedFrom where the LDS cannot hold the vectors of
// two sequences beside its area (one sequence per pass: 5.61 ms at batch 2).  A
// mixture of experts keeps the GEMV path below kMfmaBatch (its
// experts are chosen per token on that path).
constexpr int kMultiSeq = 4;
constexpr int kBatchedFrom = 2;
constexpr int kGemmBatch = 32;
constexpr int kGemmChunkK = 512;
constexpr int kActStride = kGemmChunkK + 8;   // bf16 per staged activation row (bank spread)
constexpr int kGemmMaxBlk = 4;            // 16-row blocks per wave per pass over the weights
constexpr int kMaxKSlices = 16;           // K slices of a batched product (partial sums)
constexpr int kGemmResidentK = 2 * kGemmChunkK;   // K columns a workgroup keeps resident
// LDS of the batched path (bytes): two activation chunks of both terms, and
// per-wave weight re-layout slots (2 KiB)
constexpr int kGemmActBytes = kGemmBatch * kActStride * 2;   // one term of one chunk
constexpr int kGemmLdsBytes = 4 * kGemmActBytes + kWaves * 2048;
constexpr int kNormCntStride = 64;        // words between batched RMSNorm slice counters
constexpr int kDownGather = 8;            // tagged words per control-wave lane per gather round
constexpr int kBarGroups = kSyncBarGroups;   // first level of the grid barrier
constexpr int kBarBytes = 8192;           // barrier counters: kBarGroups lines of 256 B
constexpr int kMaxOParts = 4;             // parts of the heads in a shared O projection
constexpr int kLdsMost = 160 * 1024;      // bytes of LDS a step may take
constexpr int kMaxHiddenVec = 39660;      // largest 2 Hp + head_dim that is taken

// FFN column blocks: the largest divisor of the k-tile count of ffn_dim that
// is at most 32 (and at most the grid).
inline int largest_divisor_at_most(int n, int cap) {
    for (int k = std::min(n, cap); k > 1; --k)
        if (n % k == 0) return k;
    return 1;
}

// K slices of a batched product over n K units of t k-tiles each, for a
// matrix of nblk 16-row blocks: the fewest slices (a divisor of n, at most
// kMaxKSlices) whose K range stays resident in LDS and that give every
// workgroup kWaves blocks or more; failing that, the resident choice with the
// most blocks per workgroup; if no slice fits in LDS, the most slices (the
// activations then stream through LDS in chunks).
inline int batched_k_slices(int n, int t, int nblk, int nwg) {
    int best = -1;
    for (int s = 1; s <= std::min(n, kMaxKSlices); ++s) {
        if (n % s || (n / s) * t * kTileK > kGemmResidentK) continue;
        best = s;
        if ((long long)nblk * s >= (long long)kWaves * nwg) break;
    }
    return best > 0 ? best : largest_divisor_at_most(n, kMaxKSlices);
}
// K slices of the gate/up and q/k/v products, whose K-slice partial sums a
// grid-wide fold reads back (the SwiGLU fold, the q/k/v fold): the fewest
// slices (a divisor of n, at most kMaxKSlices) whose K range is at most two
// resident ranges (the activations then stream through LDS) and that give
// every workgroup kWaves / 2 blocks or more; failing that, batched_k_slices.
// Fewer slices halve what the fold reads.  (8B shape, batch 32: 7.95 ms with
// 4 gate/up and 8 q/k/v slices, 7.48 with 2 and 4; the same for the O and
// down products, whose partials the next RMSNorm folds, gained nothing.)
inline int folded_k_slices(int n, int t, int nblk, int nwg) {
    for (int s = 1; s <= std::min(n, kMaxKSlices); ++s) {
        if (n % s || (n / s) * t * kTileK > 2 * kGemmResidentK) continue;
        if ((long long)nblk * s >= (long long)(kWaves / 2) * nwg) return s;
    }
    return batched_k_slices(n, t, nblk, nwg);
}
// Whether the batched O and down products (nblk 16-row blocks each, KSo and
// KSd slices) give every workgroup kWaves / 2 blocks or more.
inline bool matrix_cores_fill(int nblk, int KSo, int KSd, int nwg) {
    return (long long)nblk * std::min(KSo, KSd) >= (long long)(kWaves / 2) * nwg;
}

// Dynamic LDS layout of the step kernel (offsets in floats): the activation
// vector / attention area, the GEMV wave partials, 64 floats of small
// reductions and flags, then the barrier bases.
struct LdsLayout {
    int multi;          // sequences that share a GEMV pass, at most (1: none do)
    int mm;             // its slots on the matrix cores (0: on the vector units)
    int batched_from;   // first batch of the matrix-core path
    int red, red_seq;   // GEMV partial sums: matrix-core path, per-sequence path
    int sm, bar;
    int bytes;
};
inline bool lds_fits(const LdsLayout &s) { return s.bytes <= kLdsMost; }

// Heads that the O projection stages at a time: all, or the largest of up to
// kMaxOParts equal parts whose outputs of n sequences fit in 'area' floats.
inline int o_heads_for(const kl_config &c, int n, int area) {
    int p = 1;
    while (p < kMaxOParts && n * ((c.n_heads + p - 1) / p) * c.head_dim > area) ++p;
    return (c.n_heads + p - 1) / p;
}

// 'fills': the matrix-core path's products have blocks for the waves of the
// whole grid (matrix_cores_fill).
inline LdsLayout lds_layout_for(const kl_config &c, const Geometry &G, int own_max, bool fills) {
    const int g = c.n_heads / c.n_kv_heads, d = c.head_dim;
    // attention: two sets of queries, waves' (max, sum, output) per head, new
    // key and value; flags
    const int attn_main = 3 * g * (d + 8) + 4 * kWaves * g + 2 * kWaves * g * (d + 4) + 2 * d + 4;
    const auto round64 = [](int v) { return (v + 63) & ~63; };
    const int rs = kWaves * kRgBatch * kTileRows;   // one sequence's GEMV partial sums
    // per-sequence path, one sequence per GEMV pass: activations and RoPE row,
    // a SwiGLU block, the merged attention output
    const int one = round64(std::max({G.Hp + d, G.KTc * kTileK, attn_main, G.Ap}));
    // kMultiSeq sequences per pass, with 'outputs' floats of the merged
    // attention outputs at a time
    const auto multi = [&](int outputs) {
        return round64(std::max({kMultiSeq * (G.Hp + d), kMultiSeq * G.KTc * kTileK, outputs,
                                 attn_main}));
    };
    // The first batch of the matrix-core path: with several sequences per
    // GEMV pass the per-sequence path serves as many sequences (a
    // mixture of experts: up to kMfmaBatch - 1, as its routing needs).  The
    // matrix-core path's area (and its partial sums after it) may overlap
    // the per-sequence path's partial sums: a launch runs one of the two.
    // On the matrix cores a sequence's vector is three bf16 terms: where that
    // and the weight re-layout slots fit.
    const int mm = round64(std::max({multi(kMultiSeq * G.Ap), 3 * kMultiSeq * (G.Hp + 8) / 2 + kMultiSeq * d,
                                     3 * kMultiSeq * (G.Ap + 8) / 2,
                                     3 * kMultiSeq * (G.KTc * kTileK + 8) / 2}));
    // (n sequences per pass)
    const auto layout = [&](int n, int outputs, bool use_mm) {
        LdsLayout s{};
        s.multi = n;
        s.mm = use_mm ? mm : 0;
        s.batched_from = c.n_experts > 1 ? kMfmaBatch : (n > 1 ? n + 1 : kBatchedFrom);
        const int seq_a = use_mm ? mm + kWaves * 2048 / 4 : (n > 1 ? multi(outputs) : one);
        const int seq_end = seq_a + n * rs;
        const bool bat = c.max_batch >= s.batched_from;
        const int bat_a = bat ? round64(std::max(seq_a, kGemmLdsBytes / 4)) : seq_a;
        s.red_seq = seq_a;
        s.red = bat_a;
        s.sm = std::max(seq_end, bat_a + rs);
        s.bar = s.sm + 64;
        // + the step's epoch, position and validity per sequence, the experts
        // and their weights per sequence (two slots), the workgroup's share of
        // the attention, the head's argmax keys of a group of sequences and,
        // per-sequence path, the workgroup's residual rows (over the keys of
        // the matrix-core path's larger groups)
        const int seqs = std::min(c.max_batch, s.batched_from - 1);
        s.bytes = (s.bar + 2 * kBarGroups + 4 + 2 * kMfmaBatch + 4 * kMfmaBatch + 8 +
                   2 * std::max(kMfmaBatch + seqs * own_max, kGemmBatch)) * (int)sizeof(float);
        return s;
    };
    if (c.max_batch >= 2) {
        // Many heads: the attention outputs of kMultiSeq sequences do not fit
        // in LDS.  Where the matrix-core path's products fill the waves it
        // takes the batches whose outputs do not fit; elsewhere, and with
        // experts, kMultiSeq sequences share the pass a part of the heads at a
        // time, with LDS for all heads of as many as fit.  8 layers, contexts
        // 1000, us (all heads | in parts | matrix-core path):
        //   hidden 5120, 80 heads of 128, ffn 13824 (fills), batch 2:
        //     1253 | 1287 | 1348; 3: 1358 | 1382 | 1355; 4: - | 1520 | 1381;
        //   hidden 6144, 96 heads, ffn 16384 (fills), batch 2: 1560 | 1602 |
        //     1700; 3: 1674 | 1690 | 1650; 4: - | 1815 | 1720;
        //   hidden 5120, 160 heads (fills), batch 2: - | 1637 | 1601;
        //   hidden 2560, 72 heads, ffn 9728 (one K slice of the down product:
        //     160 blocks in all), batch 2: 733 | 764 | 1186; 3: 814 | 860 |
        //     1245; 4: - | 942 | 1204.
        LdsLayout s = layout(kMultiSeq, kMultiSeq * G.Ap, true);
        if (!lds_fits(s)) s = layout(kMultiSeq, kMultiSeq * G.Ap, false);
        if (!lds_fits(s) && fills && c.n_experts <= 1) s = layout(2, 2 * G.Ap, false);
        else if (!lds_fits(s)) {
            for (int n = kMultiSeq - 1; !lds_fits(s) && n >= 2; --n)
                if (kMultiSeq * ((c.n_heads + kMaxOParts - 1) / kMaxOParts) * d <= n * G.Ap)
                    s = layout(kMultiSeq, n * G.Ap, false);
            for (int p = 2; !lds_fits(s) && p <= kMaxOParts; ++p)
                s = layout(kMultiSeq, kMultiSeq * ((c.n_heads + p - 1) / p) * d, false);
        }
        if (lds_fits(s)) return s;
    }
    return layout(1, 0, false);
}

}  // namespace kl
