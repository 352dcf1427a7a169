"""Rows split over several workgroups (few query tiles against many keys): parity with the oracle,
and the same output from every entry point."""

import math
from dataclasses import replace

import numpy as np
import pytest

from gpu_util import MAX_ABS, REL_L2, compare_rows, log, to_dev
from oracle import routed_attention_rows
from synth import make_qkv, make_route_bits, pack_route_bits, small_workload, MaskSpec

CASES = [
    # B, Hq, Hk, d, L_q, L_k, block_m, causal, g
    (1, 2, 2, 64, 1024, 1024, 64, True, 1),       # short rows stay whole beside split ones
    (2, 4, 1, 128, 200, 3001, 128, True, 3),      # ragged rows and keys, odd split bounds
    (1, 1, 1, 128, 40, 20000, 64, False, 2),      # the most splits
    (1, 3, 1, 64, 1100, 900, 128, True, 1),       # rows that see no key
    (1, 2, 1, 128, 129, 4097, 128, True, 70),     # one query row and one key past the tiles
    (1, 2, 1, 128, 980, 1024, 128, True, 1),      # splits of 2 tiles; one row's tile 0 is masked for its first query
]


def _params(tm, B, Hq, Hk, d, Lq, Lk, bm, causal, g):
    return tm.Params(B, Hq, Hk, Lq, Lk, d, bm, 64, g, causal)


def test_split_scratch_is_bounded():
    """What the partial results add to the workspace, over the range of sizes: never more than the
    array tilemix_prefill_noalloc keeps for them, nothing from 1025 rows on, and for every case
    above more than nothing."""
    import paper_2608_17336_amd as tm
    bound = 1024 * (128 * 128 * 4 + 4 * 64 * 2 * 4) + 512
    rng = np.random.default_rng(5)
    for _ in range(400):
        lk = int(2 ** rng.uniform(0, 18))
        hk = int(rng.integers(1, 9))
        p = tm.Params(int(rng.integers(1, 5)), hk * int(rng.integers(1, 9)), hk, int(2 ** rng.uniform(0, 17)), lk,
                      int(rng.choice([64, 128])), int(rng.choice([64, 128])), 64, 1, bool(rng.integers(2)))
        extra = tm.tilemix_workspace_size(p) - tm.tilemix_workspace_size(replace(p, len_q=1025 * 128))
        rows = p.batch * p.heads_q * p.T_m
        assert 0 <= extra <= bound and (extra == 0 or rows <= 512), (p, extra)
    for case in CASES:
        p = _params(tm, *case)
        assert tm.tilemix_workspace_size(p) > tm.tilemix_workspace_size(replace(p, len_q=1025 * 128)), p


@pytest.mark.parametrize("whole,B,Hq,Hk,d,Lq,Lk,bm,causal", [
    # 528 to 768 pieces of one size where 512 run at once: two rounds (64.3 us against 48.2 whole; 79.5, 68.0;
    # 114.8, 100.2; 123.9, 112.8)
    (True, 1, 8, 2, 128, 2058, 2058, 64, False), (True, 1, 28, 4, 128, 700, 3000, 64, False),
    (True, 8, 2, 2, 128, 2098, 4076, 128, False), (True, 8, 1, 1, 128, 4528, 4528, 128, False),
    # short rows of d = 64, whose tiles cost less (40.0, 36.0; 27.9, 24.3; 42.1, 37.7)
    (True, 1, 32, 8, 64, 2048, 2048, 128, True), (True, 4, 8, 8, 64, 1122, 1122, 128, True),
    (True, 1, 28, 4, 64, 2170, 2170, 128, True),
    # calls that gain (95.4, 113.3; 102, 162; 68.6, 141.5; 62.7, 82.6; 14.1, 19.7; 34.9, 54.5)
    (False, 1, 8, 2, 128, 6000, 6000, 128, True), (False, 2, 16, 4, 128, 500, 9777, 128, True),
    (False, 4, 16, 4, 128, 128, 8000, 128, False), (False, 1, 8, 2, 64, 6000, 6000, 128, True),
    (False, 1, 2, 2, 64, 1024, 1024, 64, True), (False, 2, 2, 2, 64, 3848, 3848, 64, True),
])
def test_rows_are_split_where_it_pays(whole, B, Hq, Hk, d, Lq, Lk, bm, causal):
    """Calls measured with and without split rows (us in the comments): no split scratch in the workspace
    of those that are faster whole."""
    import paper_2608_17336_amd as tm
    p = _params(tm, B, Hq, Hk, d, Lq, Lk, bm, causal, 1)
    assert (tm.tilemix_workspace_size(p) == _base_bytes(tm, p)) == whole


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hk,d,Lq,Lk,bm,causal,g", CASES, ids=[str(c) for c in CASES])
def test_split_rows_parity(B, Hq, Hk, d, Lq, Lk, bm, causal, g):
    import torch
    import paper_2608_17336_amd as tm
    cfg = small_workload("split", B=B, Hq=Hq, Hk=Hk, d=d, L=max(Lq, Lk), block_m=bm, group_size=g,
                         k_outliers=True, causal=causal, index=1500 + Lq)
    Q, K, V = make_qkv(cfg)
    Q, K, V = Q[:, :Lq], K[:, :Lk], V[:, :Lk]
    rng = np.random.default_rng(Lk)
    T_mask = -(-(-(-Lk // 64)) // g)
    words = pack_route_bits((rng.random((Hk, -(-Lq // bm), T_mask)) < 0.6).astype(np.uint8))
    q, k, v, w = to_dev(Q), to_dev(K), to_dev(V), to_dev(words)
    args = (w, g, (bm, 64), causal, cfg.scale)
    log(f"split {B=} {Hq=} {Lq=} {Lk=}")
    O = tm.tilemix_prefill(q, k, v, *args)
    rows = [(b, h, np.arange(Lq)) for b in range(B) for h in range(Hq)]
    ref = routed_attention_rows(Q, K, V, words, block_m=bm, block_n=64, group_size=g, causal=causal,
                                scale=cfg.scale, rows=rows)
    mx, rel = compare_rows(O, rows, ref)
    log(f"  max_abs={mx:.3e} rel_l2={rel:.3e}")
    assert mx <= MAX_ABS and rel <= REL_L2, (mx, rel)
    same = lambda x: bool(torch.equal(x.view(torch.int16), O.view(torch.int16)))   # noqa: E731
    for again in range(2):
        assert same(tm.tilemix_prefill(q, k, v, *args)), again
    assert same(tm.tilemix_prefill_fused(q, k, v, *args))
    out = torch.full_like(O, float("nan"))
    assert same(tm.tilemix_prefill_noalloc(q, k, v, *args, O=out))
    # A workspace without room for partial results, and the attend entry point: one workgroup a row.
    p = _params(tm, B, Hq, Hk, d, Lq, Lk, bm, causal, g)
    small = torch.empty(tm.tilemix_workspace_size(replace(p, len_q=1025 * 128)), dtype=torch.uint8, device="cuda")
    whole = tm.tilemix_prefill(q, k, v, *args, workspace=small)
    mx, rel = compare_rows(whole, rows, ref)
    assert mx <= MAX_ABS and rel <= REL_L2, (mx, rel)
    ws = tm.tilemix_prepare(q, k, v, *args[1:])
    att = tm.tilemix_attend(q, k, w, ws, *args[1:])
    assert torch.equal(att.view(torch.int16), whole.view(torch.int16))
    with pytest.raises(ValueError):
        tm.tilemix_prefill(q, k, v, *args, workspace=small[:-512])


def _base_bytes(tm, p, fused=False):
    """Workspace of a call that runs one workgroup per row (1025 rows are never split)."""
    size = tm.tilemix_fused_workspace_size if fused else tm.tilemix_workspace_size
    return size(replace(p, len_q=1025 * 128))


@pytest.mark.gpu
@pytest.mark.parametrize("fused", [False, True], ids=["quantize-once", "fused"])
@pytest.mark.parametrize("B,Hq,Hk,d,Lq,Lk,bm,causal,g", CASES, ids=[str(c) for c in CASES])
def test_split_and_whole_rows_round_p_alike(B, Hq, Hk, d, Lq, Lk, bm, causal, g, fused):
    """Every workgroup of a split row starts its running max at the row's tile 0, as a whole row does, so
    both sum the same FP16 P and only the order of the FP32 sums differs.  That moves few outputs
    across a rounding boundary of FP16 (0.04 to 0.2 percent of them here); a P that is rounded
    relative to another maximum moves a quarter to half of them."""
    import torch
    import paper_2608_17336_amd as tm
    rng = np.random.default_rng(Lq + Lk)
    q, k, v = (to_dev(rng.standard_normal((B, L, H, d)).astype(np.float16))
               for L, H in ((Lq, Hq), (Lk, Hk), (Lk, Hk)))
    T_mask = -(-(-(-Lk // 64)) // g)
    w = to_dev(pack_route_bits((rng.random((Hk, -(-Lq // bm), T_mask)) < 0.5).astype(np.uint8)))
    args = (w, g, (bm, 64), causal, d ** -0.5)
    call = tm.tilemix_prefill_fused if fused else tm.tilemix_prefill
    p = _params(tm, B, Hq, Hk, d, Lq, Lk, bm, causal, g)
    split = call(q, k, v, *args)
    whole = call(q, k, v, *args, workspace=torch.empty(_base_bytes(tm, p, fused), dtype=torch.uint8, device="cuda"))
    differ = (split != whole).float().mean().item()
    log(f"split against whole {B=} {Hq=} {Lq=} {Lk=} {fused=}: {differ:.4f} of the values differ")
    assert 0.0 < differ < 0.02


@pytest.mark.gpu
@pytest.mark.parametrize("fused", [False, True], ids=["quantize-once", "fused"])
def test_split_without_a_finite_score(fused):
    """Scores of minus infinity in all keys of several splits: those keys have probability 0, and the
    row is the attention over the others, split or whole."""
    import torch
    import paper_2608_17336_amd as tm
    Lq, Lk, d = 129, 4097, 128
    rng = np.random.default_rng(8)
    Q, K, V = (rng.standard_normal((1, L, H, d)).astype(np.float16) for L, H in ((Lq, 2), (Lk, 1), (Lk, 1)))
    Q[..., 0] = 1.0
    dead = slice(512, 3000)
    words = np.zeros((1, 1, 2, 2), np.uint64)
    live = np.r_[0:512, 3000:Lk]
    rows = [(0, h, np.arange(Lq)) for h in range(2)]
    ref = routed_attention_rows(Q, K[:, live], V[:, live], words, block_m=128, block_n=64, group_size=1,
                                causal=False, scale=d ** -0.5, rows=rows)
    K[:, dead, :, 0] = -np.inf
    args = (to_dev(words), 1, (128, 64), False, d ** -0.5)
    call = tm.tilemix_prefill_fused if fused else tm.tilemix_prefill
    p = tm.Params(1, 2, 1, Lq, Lk, d, causal=False)
    base = torch.empty(_base_bytes(tm, p, fused), dtype=torch.uint8, device="cuda")
    for workspace in (None, base):
        O = call(to_dev(Q), to_dev(K), to_dev(V), *args, workspace=workspace)
        mx, rel = compare_rows(O, rows, ref)
        log(f"no finite score, split={workspace is None}: max_abs={mx:.3e} rel_l2={rel:.3e}")
        assert mx <= MAX_ABS and rel <= REL_L2, (mx, rel)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hk,L,causal", [(16, 4, 2100, True), (16, 4, 2100, False), (6, 3, 11000, True)])
def test_two_heads_per_workgroup(Hq, Hk, L, causal):
    """64-row tiles of d = 128 with an even GQA group and more than 512 tiles: two heads share a
    workgroup.  Bit for bit the one-head kernel (which exports its operands), the fused mode alike,
    and sampled rows of a pair's both heads against the oracle."""
    import torch
    import paper_2608_17336_amd as tm
    cfg = small_workload("pair", B=1, Hq=Hq, Hk=Hk, d=128, L=L, block_m=64, group_size=5, k_outliers=True,
                         causal=causal, index=1600 + L)
    Q, K, V = make_qkv(cfg)
    words, _ = make_route_bits(cfg, MaskSpec("bernoulli", 0.5))
    q, k, v, w = to_dev(Q), to_dev(K), to_dev(V), to_dev(words)
    args = (w, 5, (64, 64), causal, cfg.scale)
    log(f"two heads {Hq=} {Hk=} {L=} {causal=}")
    O = tm.tilemix_prefill(q, k, v, *args)
    if L < 4000:   # (the export of every tile product would take 5 GB for the longer case)
        one = tm.tilemix_debug_prefill(q, k, v, *args)[0]
        assert torch.equal(one.view(torch.int16), O.view(torch.int16))
    fused = tm.tilemix_prefill_fused(q, k, v, *args)
    assert torch.equal(fused.view(torch.int16), O.view(torch.int16))
    idx = np.unique(np.concatenate([np.arange(3), np.arange(60, 70), np.arange(120, 130),
                                    np.arange(L - 70, L), np.random.default_rng(L).integers(0, L, 60)]))
    rows = [(0, h, idx) for h in (0, 1, Hq // Hk, Hq - 2, Hq - 1)]
    ref = routed_attention_rows(Q, K, V, words, block_m=64, block_n=64, group_size=5, causal=causal,
                                scale=cfg.scale, rows=rows)
    mx, rel = compare_rows(O, rows, ref)
    log(f"  max_abs={mx:.3e} rel_l2={rel:.3e}")
    assert mx <= MAX_ABS and rel <= REL_L2, (mx, rel)


def _both_paths(tm, p, fused):
    """Workspaces of one call: its rows split, and one workgroup a row (with the main loop over all of its
    tiles, as every large prefill and tilemix_attend run it)."""
    import torch
    full = (tm.tilemix_fused_workspace_size if fused else tm.tilemix_workspace_size)(p)
    base = _base_bytes(tm, p, fused)
    assert base < full, p
    for label, nbytes in (("split", full), ("whole", base)):
        yield label, torch.empty(nbytes, dtype=torch.uint8, device="cuda")


FUSED = pytest.mark.parametrize("fused", [False, True], ids=["quantize-once", "fused"])


@pytest.mark.gpu
@FUSED
def test_running_max_refreshes_split_and_whole(fused):
    """Keys whose norm grows along the sequence: a whole row refreshes its running max, and rescales, many
    times in its loop; a workgroup of a split row a few times."""
    import paper_2608_17336_amd as tm
    cfg = small_workload("refresh", B=1, Hq=4, Hk=2, d=128, L=1024, block_m=128, group_size=1, k_outliers=True,
                         index=1710)
    Q, K, V = make_qkv(cfg)
    K = (K.astype(np.float32) * (1.0 + np.arange(cfg.L, dtype=np.float32) / 48.0)[None, :, None, None]).astype(np.float16)
    call = tm.tilemix_prefill_fused if fused else tm.tilemix_prefill
    rows = [(0, h, np.arange(cfg.L)) for h in range(cfg.Hq)]
    for mask in (MaskSpec("bernoulli", 0.5), MaskSpec("all_fp16"), MaskSpec("all_int8")):
        words, _ = make_route_bits(cfg, mask)
        ref = routed_attention_rows(Q, K, V, words, block_m=128, block_n=64, group_size=1, causal=True,
                                    scale=cfg.scale, rows=rows)
        p = _params(tm, 1, 4, 2, 128, cfg.L, cfg.L, 128, True, 1)
        for label, ws in _both_paths(tm, p, fused):
            O = call(to_dev(Q), to_dev(K), to_dev(V), to_dev(words), 1, (128, 64), True, cfg.scale, workspace=ws)
            mx, rel = compare_rows(O, rows, ref)
            log(f"refresh {mask.label} {label} {fused=}: max_abs={mx:.3e} rel_l2={rel:.3e}")
            assert mx <= MAX_ABS and rel <= REL_L2, (mask.label, label, mx, rel)


@pytest.mark.gpu
@FUSED
def test_fold_bound_passed_in_the_loop(fused):
    """INT8 tiles whose biased start is admitted against the running max as it stands, and a score jump
    that moves it past the fold's bound in the middle of the row: the bias is dropped from the
    affected tiles, and those after it start at 0."""
    import paper_2608_17336_amd as tm
    rng = np.random.default_rng(11)
    d, L, scale = 128, 1024, 1.0 / math.sqrt(128)
    u = np.where(rng.random(d) < 0.5, -1.0, 1.0).astype(np.float32)
    s_k = np.where(np.arange(L // 64) < 9, 25.0, 36.25)   # log2 scores of about 1630, then 2365
    Q = (4.0 * np.tile(u, (L, 1)))[None, :, None, :].astype(np.float16)
    K = (np.repeat(s_k, 64)[:, None] * u[None, :])[None, :, None, :].astype(np.float16)
    V = rng.standard_normal((1, L, 1, d), dtype=np.float32).astype(np.float16)
    words = pack_route_bits(np.ones((1, L // 128, L // 64), np.uint8))
    rows = [(0, 0, np.arange(L))]
    ref = routed_attention_rows(Q, K, V, words, block_m=128, block_n=64, group_size=1, causal=True, scale=scale,
                                rows=rows)
    call = tm.tilemix_prefill_fused if fused else tm.tilemix_prefill
    for label, ws in _both_paths(tm, _params(tm, 1, 1, 1, d, L, L, 128, True, 1), fused):
        O = call(to_dev(Q), to_dev(K), to_dev(V), to_dev(words), 1, (128, 64), True, scale, workspace=ws)
        mx, rel = compare_rows(O, rows, ref)
        log(f"fold bound {label} {fused=}: max_abs={mx:.3e} rel_l2={rel:.3e}")
        assert mx <= MAX_ABS and rel <= REL_L2, (label, mx, rel)


@pytest.mark.gpu
@FUSED
def test_integer_inputs_split_and_whole(fused):
    """Inputs whose codes are the inputs (every block's absmax is 127): with exactly converted products the
    routes agree bit for bit, also where the running max is refreshed again and again."""
    import torch
    import paper_2608_17336_amd as tm
    rng = np.random.default_rng(9)
    L = 1024
    Q = rng.integers(-127, 128, size=(1, L, 4, 128)).astype(np.float16)
    K = rng.integers(-127, 128, size=(1, L, 2, 128)).astype(np.float16)
    Q[:, ::128, :, 0] = 127.0
    K[:, ::64, :, 0] = -127.0
    V = rng.standard_normal((1, L, 2, 128)).astype(np.float16)
    q, k, v = to_dev(Q), to_dev(K), to_dev(V)
    call = tm.tilemix_prefill_fused if fused else tm.tilemix_prefill
    p = _params(tm, 1, 4, 2, 128, L, L, 128, True, 1)
    for label, ws in _both_paths(tm, p, fused):
        routes = [call(q, k, v, to_dev(pack_route_bits(np.full((2, L // 128, L // 64), bit, np.uint8))), 1, (128, 64),
                       True, 1.0 / 512.0, workspace=ws) for bit in (0, 1)]
        log(f"integer inputs {label} {fused=}")
        assert torch.equal(routes[0].view(torch.int16), routes[1].view(torch.int16)), label


@pytest.mark.gpu
def test_longest_row_split_and_whole():
    """L_k = 262144: 4096 tiles in one workgroup (all its key scales, routing words and the 64-tile ring of
    routes), against 64 splits; the fused mode bit for bit alike on either path."""
    import torch
    import paper_2608_17336_amd as tm
    rng = np.random.default_rng(262146)
    Lq, Lk, d = 200, 262144, 128
    q, k, v = (to_dev(rng.standard_normal((1, L, H, d)).astype(np.float16)) for L, H in ((Lq, 2), (Lk, 1), (Lk, 1)))
    w = to_dev(pack_route_bits((rng.random((1, 2, Lk // 64)) < 0.5).astype(np.uint8)))
    p = _params(tm, 1, 2, 1, d, Lq, Lk, 128, True, 1)
    outs = {}
    for fused in (False, True):
        call = tm.tilemix_prefill_fused if fused else tm.tilemix_prefill
        for label, ws in _both_paths(tm, p, fused):
            log(f"longest row {label} {fused=}")
            outs[label, fused] = call(q, k, v, w, 1, (128, 64), True, d ** -0.5, workspace=ws)
    for label in ("split", "whole"):
        assert torch.equal(outs[label, False].view(torch.int16), outs[label, True].view(torch.int16)), label
    a, b = outs["split", False], outs["whole", False]
    differ = (a != b).float().mean().item()
    log(f"  {differ:.4f} of the values differ")
    # the same P (see above) and FP32 sums of 262144 terms in another order
    assert differ < 0.1 and torch.allclose(a.float(), b.float(), rtol=2 ** -10, atol=1e-5)
