"""The attention's shares (equal runs of 4 KiB units of the batch's cached
positions, or whole workgroups per sequence) and the hand-offs by row owner, at
the places where they can go wrong: empty contexts, contexts around a unit
(16 positions at head dimension 128, 32 at 64), fewer units than workgroups,
more sequences than workgroups per KV head, sequences split over many shares,
rows that do not divide the grid.  Against the oracle, every schedule bit for
bit the same.  The bounds are those of the other parity tests."""
import numpy as np
import pytest

from paper_2410_23668_amd import binding as kb
from synth.workloads import TINY
from tests.gpu_cases import MODES, Case, assert_bit_exact, check_against_oracle, say

pytestmark = pytest.mark.gpu

D64 = dict(TINY, n_layers=2)
D128 = dict(TINY, n_layers=2, head_dim=128, hidden=264, ffn_dim=200)
MHA = dict(TINY, n_layers=2, n_heads=64, n_kv_heads=64)      # 4 workgroups per KV head
G8 = dict(D128, n_heads=16, n_kv_heads=2)

CASES = [
    ("d64 one", D64, [0]),
    ("d64 units", D64, [31, 32, 33]),
    ("d64 batched units", D64, [0, 1, 31, 32, 63, 64, 65, 500]),
    ("d128 one", D128, [0]),
    ("d128 units", D128, [15, 16, 17, 0]),
    ("d128 long and short", D128, [3000, 1]),
    ("d128 batched long and short", D128, [0, 2900, 16, 15, 1, 800]),
    ("4 workgroups per head", MHA, [70, 0, 33]),
    ("one long context, 4 workgroups per head", MHA, [3000, 10, 3, 40]),
    ("one long context, 128 workgroups per head", D128, [3, 2500, 40]),
    ("more sequences than workgroups per head", MHA, [5, 64, 0, 31, 200, 1, 32]),
    ("2 workgroups per head", dict(MHA, n_heads=128, n_kv_heads=128), [40, 0, 100]),
    ("8 heads per KV head", G8, [1000, 17]),
    ("8 heads per KV head, batched", G8, [40, 0, 777, 16, 15]),
    ("33 sequences", D128, [(37 * i) % 130 for i in range(33)]),
]


@pytest.mark.parametrize("name,cfg,filled", CASES, ids=[c[0] for c in CASES])
def test_shares_of_the_attention(name, cfg, filled):
    say(f"[shares] {name}: contexts {filled}")
    cap = (max(filled) + 1 + 63) // 64 * 64
    c = Case(cfg, len(filled), cap, np.asarray(filled, dtype=np.int32), seed=311 + len(filled))
    ref = c.oracle_step(nthreads=8)
    outs = [c.gpu_step(mode) for _, mode in MODES]
    check_against_oracle(c, outs[1], ref)
    for (what, _), o in zip(MODES, outs):
        assert_bit_exact(o, outs[1], f"{what} vs looped")
    assert c.model.device_error() == 0
    c.model.close()


@pytest.mark.parametrize("hidden,batch", [(256, 6), (1032, 5), (520, 37)])
def test_swiglu_in_the_gate_up_epilogue(hidden, batch):
    """An FFN wide enough for one K slice of the batched gate/up product (the
    SwiGLU is applied to its products directly): activations resident in LDS
    (256, 520 columns) and streamed (1032), a second group of sequences (37)."""
    cfg = dict(TINY, n_layers=2, hidden=hidden, ffn_dim=13320)
    say(f"[swiglu epilogue] hidden {hidden} batch {batch}")
    filled = (np.arange(batch, dtype=np.int32) * 29 + 3) % 90
    c = Case(cfg, batch, 128, filled, seed=411 + batch)
    ref = c.oracle_step(nthreads=8, sample=[0, batch // 2, batch - 1])
    outs = [c.gpu_step(mode) for _, mode in MODES]
    check_against_oracle(c, outs[1], ref, only=[0, batch // 2, batch - 1])
    for (what, _), o in zip(MODES, outs):
        assert_bit_exact(o, outs[1], f"{what} vs looped")
    c.model.close()


@pytest.mark.parametrize("over,batch", [
    (dict(hidden=64, ffn_dim=72), 2),                  # one tile of columns: whole row groups per wave
    (dict(hidden=264, ffn_dim=200), 4),
    (dict(hidden=1032, ffn_dim=3000), 3),              # column slices of uneven length, a padded one
    (dict(hidden=1040, ffn_dim=1096, head_dim=128), 2),
    (dict(hidden=520, ffn_dim=264, n_experts=4, top_k=2), 3),
    (dict(hidden=6152, ffn_dim=520), 3),               # too wide for LDS: the vector-unit form
    # heads whose outputs do not fit in LDS for all sequences: the O projection
    # in 2 or 3 parts of them, or (matrix cores busy from batch 4 on) in one
    (dict(hidden=264, head_dim=128, n_heads=72, n_kv_heads=9, ffn_dim=200), 4),
    (dict(hidden=2560, n_heads=150, n_kv_heads=75, ffn_dim=264), 4),
    (dict(hidden=520, head_dim=128, n_heads=200, n_kv_heads=25, ffn_dim=264), 3),
    (dict(hidden=4096, head_dim=128, n_heads=128, n_kv_heads=16, ffn_dim=264), 2),
    (dict(hidden=264, head_dim=128, n_heads=72, n_kv_heads=9, ffn_dim=200, n_experts=4, top_k=2), 4),
], ids=str)
def test_sequences_sharing_a_pass(over, batch):
    """Batches of 2 to 4 take each weight pass together: on the matrix cores
    (three bf16 terms of each vector) where LDS holds the terms, else on the
    vector units."""
    cfg = dict(TINY, n_layers=2, **over)
    say(f"[shared pass] {over} batch {batch}")
    filled = (np.arange(batch, dtype=np.int32) * 29 + 3) % 90
    c = Case(cfg, batch, 128, filled, seed=511 + batch)
    # (not one sequence per pass, nor the matrix-core path from batch 2 on)
    want = 8 if "n_experts" in over else (3 if over.get("n_heads") == 128 else 5)
    assert c.model.info().mfma_min_batch == want
    ref = c.oracle_step(nthreads=8)
    # (a mixture of experts has no per-op schedule)
    modes = [m for m in MODES if not ("n_experts" in over and m[1] == kb.KL_MODE_PER_OP)]
    outs = {what: c.gpu_step(mode) for what, mode in modes}
    check_against_oracle(c, outs["looped"], ref)
    for what, o in outs.items():
        assert_bit_exact(o, outs["looped"], f"{what} vs looped")
    assert c.model.device_error() == 0
    c.model.close()


@pytest.mark.parametrize("over,batch", [
    # K slices of 384 columns (gate/up), resident
    (dict(hidden=768, ffn_dim=4096), 5),
    # 8 K slices of 320 columns (q/k/v), resident
    (dict(hidden=2560, n_heads=16, n_kv_heads=4, head_dim=128, ffn_dim=264), 6),
    # 4 K slices of 1280 columns (q/k/v), streamed through LDS
    (dict(hidden=5120, n_heads=28, n_kv_heads=14, head_dim=128, ffn_dim=264), 5),
], ids=str)
def test_k_slices_across_the_slices_of_the_norm(over, batch):
    """K slices that do not start on a slice of the RMSNorm hand-off (512
    columns): a staged chunk lies in two of them and waits for both."""
    cfg = dict(TINY, n_layers=2, **over)
    say(f"[straddling slices] {over} batch {batch}")
    filled = (np.arange(batch, dtype=np.int32) * 29 + 3) % 90
    c = Case(cfg, batch, 128, filled, seed=611 + batch)
    ref = c.oracle_step(nthreads=8, sample=[0, batch - 1])
    outs = [c.gpu_step(mode) for _, mode in MODES]
    check_against_oracle(c, outs[1], ref, only=[0, batch - 1])
    for (what, _), o in zip(MODES, outs):
        assert_bit_exact(o, outs[1], f"{what} vs looped")
    assert c.model.device_error() == 0
    c.model.close()


@pytest.mark.parametrize("hidden,batch,experts", [(19776, 1, 0), (9024, 4, 0), (19776, 7, 4),
                                                  (9024, 3, 4)])
def test_hidden_sizes_that_fill_lds(hidden, batch, experts):
    """The largest hidden size, and the largest whose sequences share a pass:
    LDS has to hold the residual rows that a workgroup owns as well."""
    cfg = dict(TINY, n_layers=3, hidden=hidden, ffn_dim=264)
    if experts:
        cfg.update(n_experts=experts, top_k=2)
    say(f"[full LDS] hidden {hidden} batch {batch} experts {experts}")
    filled = (np.arange(batch, dtype=np.int32) * 29 + 3) % 90
    c = Case(cfg, batch, 128, filled, seed=711 + batch)
    assert c.model.info().mfma_min_batch == (8 if experts else (5 if batch > 1 else 2))
    ref = c.oracle_step(nthreads=8)
    modes = [m for m in MODES if not (experts and m[1] == kb.KL_MODE_PER_OP)]
    outs = {what: c.gpu_step(mode) for what, mode in modes}
    check_against_oracle(c, outs["looped"], ref)
    for what, o in outs.items():
        assert_bit_exact(o, outs["looped"], f"{what} vs looped")
    assert c.model.device_error() == 0
    c.model.close()
