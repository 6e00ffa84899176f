"""GPU parity: lpp_tree_attention against the float64 oracle (through the C ABI).

Tolerance (relative to |want| + the row's max |want|): 1e-4 for fp32 inputs,
2e-2 for bf16 inputs (fp32 softmax/accumulation, bf16 probabilities on the
matrix cores)."""
import numpy as np
import pytest
import torch

import paper_2502_06352_amd as lpp
from oracle import tree_attention
from workloads import CONFIGS, static_tree, make_attention_inputs
from gpu_common import DEV, dev, run_attention, attention_error

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


def _check(cfg, parent, att, got, seq_len=None, pairs=None):
    B, H = att["q"].shape[:2]
    assert np.all(np.isfinite(got))
    if pairs is None:
        want = tree_attention(att["q"], att["kc"], att["vc"], att["kt"], att["vt"], parent, seq_len=seq_len)
        err = attention_error(got, want)
    else:
        err = 0.0
        for b, h in pairs:
            sl = None if seq_len is None else seq_len[b:b + 1]
            want = tree_attention(att["q"][b:b + 1, h:h + 1], att["kc"][b:b + 1, h:h + 1], att["vc"][b:b + 1, h:h + 1],
                                  att["kt"][b:b + 1, h:h + 1], att["vt"][b:b + 1, h:h + 1], parent, seq_len=sl)
            err = max(err, attention_error(got[b:b + 1, h:h + 1], want))
    print(f"cfg{cfg.idx} B={B} H={H} M={cfg.M} S={att['kc'].shape[2]} Dh={cfg.Dh} {cfg.kv_dtype}: err={err:.3e}", flush=True)
    assert err <= TOL[cfg.kv_dtype]
    return err


@pytest.mark.parametrize("idx", [1, 2, 3, 4])
def test_attention_parity_configs(idx):
    cfg = CONFIGS[idx]
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    got = run_attention(lpp.Tree(parent), att, cfg)
    _check(cfg, parent, att, got)


def test_attention_parity_stress_full_size():
    # config 5 at its full size: every head of three batch items (the first, one in the middle, the
    # last) and one head of every other item
    cfg = CONFIGS[5]
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    got = run_attention(lpp.Tree(parent), att, cfg)
    pairs = [(b, h) for b in (0, 7, cfg.B - 1) for h in range(cfg.H)]
    pairs += [(b, (5 * b + 3) % cfg.H) for b in range(cfg.B) if b not in (0, 7, cfg.B - 1)]
    _check(cfg, parent, att, got, pairs=pairs)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_ragged_lengths_and_odd_shapes(dtype):
    # S not a multiple of 32, per-item lengths (one empty), odd row counts
    for (N, branching, S, H, Dh, lens) in [
        (5, (2, 2, 1), 77, 3, 64, [77, 0, 31, 33]),
        (40, (5, 3, 2, 1), 130, 2, 128, [130, 1, 64, 97]),
        (128, (8, 4, 2, 2, 1, 1, 1, 1), 45, 2, 64, [45, 7, 0, 32]),
        (16, (16,), 100, 1, 128, [100, 99, 3, 50]),
    ]:
        cfg = CONFIGS[2].scaled(N=N, branching=branching, S=S, H=H, Dh=Dh, B=4, kv_dtype=dtype)
        parent = static_tree(cfg.branching, cfg.N)
        att = make_attention_inputs(cfg)
        sl = np.array(lens, dtype=np.int32)
        got = run_attention(lpp.Tree(parent), att, cfg, seq_len=sl)
        _check(cfg, parent, att, got, seq_len=sl)


def test_attention_no_cache_and_single_row():
    cfg = CONFIGS[2].scaled(N=0, branching=(1,), S=64, H=2, B=2)
    parent = np.array([-1], dtype=np.int32)
    att = make_attention_inputs(cfg)
    got = run_attention(lpp.Tree(parent), att, cfg)
    _check(cfg, parent, att, got)
    # S = 0: only the tree keys; a root row then returns its own V row exactly (bf16 value)
    cfg = CONFIGS[2].scaled(N=9, branching=(3, 2), S=0, H=2, B=1)
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    got = run_attention(lpp.Tree(parent), att, cfg, S=0)
    _check(cfg, parent, att, got)
    assert np.array_equal(got[:, :, 0], att["vt"][:, :, 0])


def test_attention_masked_sibling_has_no_influence():
    cfg = CONFIGS[2].scaled(S=96, H=2)
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    tree = lpp.Tree(parent)
    a = run_attention(tree, att, cfg)
    att2 = dict(att)
    from workloads import bf16_bits
    kt = att["kt"].copy(); kt[:, :, 2] *= 50.0
    att2["kt"], att2["kt_bits"] = kt, bf16_bits(kt)
    b = run_attention(tree, att2, cfg)
    from oracle import ancestor_mask
    vis = ancestor_mask(parent)
    for i in range(cfg.M):
        assert np.array_equal(a[:, :, i], b[:, :, i]) == (not vis[i, 2])


def test_attention_deterministic_run_to_run():
    cfg = CONFIGS[3]
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    tree = lpp.Tree(parent)
    assert np.array_equal(run_attention(tree, att, cfg), run_attention(tree, att, cfg))


def test_attention_argument_errors():
    cfg = CONFIGS[1].scaled(Dh=32)
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    with pytest.raises(lpp.LppError) as e:
        run_attention(lpp.Tree(parent), att, cfg)
    assert e.value.status == lpp.LPP_EUNSUPPORTED


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("N,S,lens", [
    (0, 1, [1, 0]), (14, 15, [15, 1]), (15, 16, [16, 2]), (16, 17, [17, 0]), (31, 33, [16, 31]),
    (15, 240, [240, 239]), (32, 256, [256, 241]), (60, 700, [700, 513]), (127, 530, [530, 385]),
    (15, 496, [496, 0]), (15, 1100, [1100, 3]), (4, 4200, [4200, 4111])])
def test_attention_f32_tile_edges(Dh, N, S, lens):
    # row tiles of 16, key tiles of 16, rounds of 128 or 256 keys: one short, even, one over; key ranges in
    # blocks of their own, some of them empty for a short item
    branching = (6, 3, 2, 2, 1, 1) if N <= 60 else (8, 4, 2, 2, 1, 1, 1, 1)
    cfg = CONFIGS[2].scaled(N=N, branching=branching, S=S, H=3, Dh=Dh, B=2, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N) if N else np.array([-1], dtype=np.int32)
    att = make_attention_inputs(cfg)
    sl = np.array(lens, dtype=np.int32)
    _check(cfg, parent, att, run_attention(lpp.Tree(parent), att, cfg, seq_len=sl), seq_len=sl)


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("S", [150, 900])
def test_attention_f32_ignores_what_a_row_does_not_see(Dh, bad, S):
    # a masked key, and one whose weight underflows to zero, add nothing whatever their V rows hold
    cfg = CONFIGS[2].scaled(N=20, S=S, H=2, B=1, Dh=Dh, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    tree = lpp.Tree(parent)
    from oracle import ancestor_mask
    vis = ancestor_mask(parent)
    want = tree_attention(att["q"], att["kc"], att["vc"], att["kt"], att["vt"], parent)
    kt, vt = att["kt"].copy(), att["vt"].copy()
    kt[:, :, 2], vt[:, :, 2] = bad, bad
    got = run_attention(tree, dict(att, kt=kt, vt=vt), cfg)
    unseen = ~vis[:, 2]
    assert unseen.any() and attention_error(got[:, :, unseen], want[:, :, unseen]) <= TOL["f32"]
    assert np.all(np.isnan(got[:, :, ~unseen]) | np.isinf(got[:, :, ~unseen]))
    kc, vc = att["kc"].copy(), att["vc"].copy()
    kc[:, :, 5] = -1e6 * np.sign(att["q"][:, :, :1]).squeeze(2)     # row 0 gives it no weight
    vc[:, :, 5] = bad
    got = run_attention(tree, dict(att, kc=kc, vc=vc), cfg)
    keep = np.arange(S) != 5
    want = tree_attention(att["q"], att["kc"][:, :, keep], att["vc"][:, :, keep], att["kt"], att["vt"], parent)
    assert attention_error(got[:, :, :1], want[:, :, :1]) <= TOL["f32"]


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("S", [150, 1100])
def test_attention_f32_puts_infinities_where_they_belong(Dh, S):
    # V rows with infinities of either sign and NaN, seen by all rows (cache) or by some (tree): every element of
    # the output is what a sum over the keys its row sees gives, and what holds none stays as it was
    cfg = CONFIGS[2].scaled(N=20, S=S, H=2, B=1, Dh=Dh, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    tree = lpp.Tree(parent)
    from oracle import ancestor_mask
    vis = ancestor_mask(parent)
    clean = run_attention(tree, att, cfg)
    vc, vt = att["vc"].copy(), att["vt"].copy()
    vc[0, 0, 7, 3], vc[0, 0, S - 1, 4], vc[0, 0, 40, 5], vc[0, 0, 41, 5] = np.inf, -np.inf, np.inf, -np.inf
    vt[0, 1, 2, 6], vt[0, 1, 5, 6], vt[0, 1, 1, Dh - 1] = np.inf, -np.inf, np.nan
    got = run_attention(tree, dict(att, vc=vc, vt=vt), cfg)
    want = clean.astype(np.float64)
    want[0, 0, :, 3], want[0, 0, :, 4], want[0, 0, :, 5] = np.inf, -np.inf, np.nan
    want[0, 1, vis[:, 2], 6] = np.inf
    want[0, 1, vis[:, 5], 6] = np.where(vis[vis[:, 5], 2], np.nan, -np.inf)
    want[0, 1, vis[:, 1], Dh - 1] = np.nan
    odd = ~np.isfinite(want)
    assert np.array_equal(got[odd], want[odd], equal_nan=True)
    # (an element that shares its 16 bytes with one of these is summed in another order)
    assert attention_error(np.where(odd, 0, got), np.where(odd, 0, want)) <= 1e-5


def test_attention_f32_costs_two_passes_where_a_masked_key_holds_nan():
    # 96 rows of 16 heads on 1898 keys, the last row's V a NaN: 56 us against 24; done key by key it took 866
    cfg = CONFIGS[2].scaled(N=95, branching=(8, 4, 2, 2, 1, 1, 1, 1), S=1898, H=16, B=1, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N)
    att = make_attention_inputs(cfg)
    tree = lpp.Tree(parent)
    t = {n: dev(att[n]) for n in ("q", "kc", "vc", "kt", "vt")}
    out = torch.empty((1, cfg.H, cfg.M, cfg.Dh), device=DEV)
    ws = torch.empty(lpp.lpp_tree_attention_workspace(tree, 1, cfg.H, cfg.S, cfg.Dh), dtype=torch.uint8, device=DEV)

    def least():
        best = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                lpp.lpp_tree_attention(tree, lpp.LPP_F32, t["q"], t["kc"], t["vc"], t["kt"], t["vt"], None, 1, cfg.H, cfg.S,
                                       cfg.Dh, 0.0, out, ws)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b))
        return min(best)
    plain = least()
    t["vt"][:, :, -1] = float("nan")
    assert least() < 6 * plain
