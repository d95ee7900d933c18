// The step kernel's LDS layout (kl_lds.h) over many shapes: it fits, every
// phase's staged data fit before the GEMV partial sums, and the number of heads
// does not keep sequences from sharing a pass (up to kMultiSeq; two, as far as
// their attention outputs fit, where the matrix-core path fills the waves).
// Prints "lds layout OK" and exits 0, else prints the failures and exits 1.
#include <cstdio>

#include "kl_lds.h"

using namespace kl;

namespace {

int g_fail = 0;

void check(bool ok, const char *what, const kl_config &c) {
    if (ok || ++g_fail > 20) return;
    std::fprintf(stderr, "FAIL: %s: hidden %d heads %d/%d of %d ffn %d experts %d batch %d\n", what,
                 c.hidden, c.n_heads, c.n_kv_heads, c.head_dim, c.ffn_dim, c.n_experts,
                 c.max_batch);
}

constexpr int kGrid = 256;

LdsLayout layout(const kl_config &c, Geometry &G, bool fills) {
    G = layout_geometry(c, kGrid);
    return lds_layout_for(c, G, (G.o_rg + kGrid - 1) / kGrid * kTileRows, fills);
}

kl_config config(int hidden, int d, int group, int nkv, int ffn, int experts, int batch) {
    kl_config c{};
    c.n_layers = 1; c.hidden = hidden; c.n_heads = nkv * group; c.n_kv_heads = nkv;
    c.head_dim = d; c.ffn_dim = ffn; c.vocab = 1000; c.max_batch = batch; c.max_seq = 64;
    c.n_experts = experts; c.top_k = experts ? 2 : 0;
    return c;
}

void shape(int hidden, int d, int group, int ffn, int experts, int batch, bool fills) {
    Geometry G;
    const int few_heads = layout(config(hidden, d, group, 1, ffn, experts, batch), G, fills).multi;
    for (int nkv = 1; nkv * group <= kGrid; nkv += nkv < 8 ? 1 : 5) {
        const kl_config c = config(hidden, d, group, nkv, ffn, experts, batch);
        const LdsLayout s = layout(c, G, fills);
        if (!lds_fits(s)) continue;   // (refused)
        if (fills && !experts)   // (36000 floats beside 2 sequences' partial sums: 152 KiB)
            check(s.multi == few_heads || s.multi == 2 || (s.multi == 1 && 2 * G.Ap > 36000),
                  "two sequences' outputs fit", c);
        else
            check(s.multi == few_heads, "the number of heads decides the shared pass", c);
        const int nb = s.multi;
        for (int b = 2; b <= nb; ++b) {
            const int at_once = o_heads_for(c, b, s.red_seq);
            check(at_once > 0 && b * at_once * d <= s.red_seq, "attention outputs", c);
            check(!s.mm || at_once == c.n_heads, "matrix cores: all heads at once", c);
        }
        check((nb > 1 ? kMultiSeq * G.Hp : G.Hp) + d * nb <= s.red_seq,
              "residual and RoPE rows", c);
        check(nb * G.KTc * kTileK <= s.red_seq, "a SwiGLU block", c);
        check(s.red_seq + nb * kWaves * kRgBatch * kTileRows <= s.sm, "partial sums", c);
        check(!s.mm || (nb == kMultiSeq && s.mm + kWaves * 512 <= s.red_seq), "re-layout slots", c);
        if (s.mm)
            for (int K : {G.Hp, G.Ap, G.KTc * kTileK})
                check(3 * kMultiSeq * (K + 8) / 2 + (K == G.Hp ? kMultiSeq * d : 0) <= s.mm,
                      "three terms of the vectors", c);
        if (c.max_batch >= s.batched_from)
            check(kGemmLdsBytes <= 4 * s.red, "the matrix-core path's area", c);
    }
}

// The residual rows a workgroup owns, and the share of the attention, decide
// neither whether a hidden size is taken (2 Hp + d floats and 5040 bytes of
// partial sums and tables have to fit in 160 KiB less 256 bytes) nor whether
// four sequences share a pass (4 (Hp + d) floats and 17328 bytes).
void rows_do_not_count(const kl_config &c) {
    const Geometry G = layout_geometry(c, kGrid);
    const int own = (G.o_rg + kGrid - 1) / kGrid * kTileRows, d = c.head_dim, most = 163584;
    const auto round64 = [](int v) { return (v + 63) / 64 * 64; };
    for (bool fills : {false, true}) {
        const LdsLayout s = lds_layout_for(c, G, own, fills);
        check(s.bytes <= 160 * 1024 || 2 * G.Hp + d > kMaxHiddenVec, "past the LDS", c);
        if (c.max_batch == 4)   // (larger batches: the matrix-core path's area as well)
            check((4 * round64(4 * (G.Hp + d)) + 4 * 4096 + 848 <= most) == (s.multi == 4),
                  "rows decide the shared pass", c);
    }
    check((4 * round64(2 * G.Hp + d) + 4096 + 848 <= most) == (2 * G.Hp + d <= kMaxHiddenVec),
          "hidden sizes that are taken", c);
}

}  // namespace

int main() {
    for (int hidden : {64, 264, 2560, 4096, 5120, 6144, 8192, 9216, 12288, 19648})
        for (int d : {64, 128})
            for (int group : {1, 2, 4, 8})
                for (int ffn : {200, 13824, 28672})
                    for (int experts : {0, 8})
                        for (int batch : {1, 2, 4, 32})
                            for (bool fills : {false, true})
                                shape(hidden, d, group, ffn, experts, batch, fills);
    for (int hidden = 8192; hidden <= 19968; hidden += 8)
        for (int d : {64, 128})
            for (int experts : {0, 8})
                for (int batch : {1, 2, 4, 7, 32})
                    rows_do_not_count(config(hidden, d, 4, 8, 11008, experts, batch));
    if (g_fail) return 1;
    std::printf("lds layout OK\n");
    return 0;
}
