"""GPU parity: lpp_tree_attention_layers (several layers of one step in one launch; Sec. 2.1,
App. A.2) against the float64 oracle, layer by layer, through the C ABI.  Every layer has its own
queries, keys and values (seeded apart), so a block that reads another layer's tensors, partials
or counters shows up as an error."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2502_06352_amd as lpp
from oracle import tree_attention
from workloads import CONFIGS, static_tree, make_attention_inputs
from gpu_common import DEV, dev, bf16_dev, attention_error

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


def _layer_inputs(cfg, Hkv, layer):
    att = make_attention_inputs(cfg, salt=10 * layer)
    if Hkv != cfg.H:
        kv = make_attention_inputs(dataclasses.replace(cfg, H=Hkv), salt=10 * layer + 1)
        for n in ("kc", "vc", "kt", "vt"):
            att[n] = kv[n]
            if n + "_bits" in kv:
                att[n + "_bits"] = kv[n + "_bits"]
    return att


def _run_layers(tree, atts, cfg, Hkv, out_dtype=lpp.LPP_F32, seq_len=None):
    B, H, M, Dh = atts[0]["q"].shape
    S = atts[0]["kc"].shape[2]
    bf = cfg.kv_dtype == "bf16"
    names = {"q": "q", "kc": "k_cache", "vc": "v_cache", "kt": "k_tree", "vt": "v_tree"}
    layers, outs = [], []
    for att in atts:
        y = {names[n]: (bf16_dev(att[n + "_bits"]) if bf else dev(att[n])) for n in names}
        y["out"] = torch.full((B, H, M, Dh), float("nan"),
                              dtype=torch.bfloat16 if out_dtype == lpp.LPP_BF16 else torch.float32, device=DEV)
        layers.append(y)
        outs.append(y["out"])
    sl = None if seq_len is None else dev(np.asarray(seq_len, dtype=np.int32))
    L = len(layers)
    ws = torch.empty(max(lpp.lpp_tree_attention_layers_workspace(tree, L, B, H, S, Dh), 256), dtype=torch.uint8, device=DEV)
    lpp.lpp_tree_attention_layers(tree, lpp.LPP_BF16 if bf else lpp.LPP_F32, out_dtype, layers, sl, B, H, Hkv, S, Dh, 0.0, ws)
    torch.cuda.synchronize()
    return [o.float().cpu().numpy() for o in outs]


@pytest.mark.parametrize("idx,L,Hkv", [(1, 3, 4), (2, 3, 16), (3, 3, 24), (4, 3, 32), (2, 19, 16), (3, 2, 8),
                                       (4, 5, 8)])
def test_layers_parity(idx, L, Hkv):
    # cfg 2 and 4 at L = 3 split the keys of a head over several blocks (partials and counters per
    # layer); L = 19 takes two launches; cfg 3 with 8 key/value heads shares them among query heads.
    # Launches with more blocks than compute units run blocks of 4 waves: cfg 3 at L = 2 and 3
    # (head size 64), cfg 4 at L = 5 (head size 128, 8 key/value heads).
    cfg = CONFIGS[idx]
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    atts = [_layer_inputs(cfg, Hkv, l) for l in range(L)]
    got = _run_layers(tree, atts, cfg, Hkv)
    worst = 0.0
    for l in range(L):
        want = tree_attention(atts[l]["q"], atts[l]["kc"], atts[l]["vc"], atts[l]["kt"], atts[l]["vt"], parent)
        err = attention_error(got[l], want)
        worst = max(worst, err)
        assert np.all(np.isfinite(got[l])) and err <= TOL[cfg.kv_dtype], f"layer {l}: err {err}"
    print(f"cfg{idx} L={L} Hkv={Hkv}: worst err {worst:.3e}", flush=True)


def test_layers_equal_the_single_layer_call_and_repeat():
    # the same layers through lpp_tree_attention one by one: identical bits; twice on one handle
    cfg = CONFIGS[2]
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    atts = [_layer_inputs(cfg, cfg.H, l) for l in range(4)]
    a = _run_layers(tree, atts, cfg, cfg.H)
    b = _run_layers(tree, atts, cfg, cfg.H)
    from gpu_common import run_attention
    for l in range(4):
        one = run_attention(tree, atts[l], cfg)
        assert np.array_equal(a[l], b[l])
        err = attention_error(a[l], one)
        assert err <= 1e-5, f"layer {l} differs from the single-layer call by {err}"   # (other key splits: other rounding)


def test_layers_ragged_lengths_bf16_out_and_errors():
    cfg = CONFIGS[3].scaled(B=3)
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    atts = [_layer_inputs(cfg, 8, l) for l in range(2)]
    seq = [0, 517, cfg.S]
    got = _run_layers(tree, atts, cfg, 8, out_dtype=lpp.LPP_BF16, seq_len=seq)
    for l in range(2):
        for b, n in enumerate(seq):
            want = tree_attention(atts[l]["q"][b:b + 1], atts[l]["kc"][b:b + 1, :, :n], atts[l]["vc"][b:b + 1, :, :n],
                                  atts[l]["kt"][b:b + 1], atts[l]["vt"][b:b + 1], parent)
            assert attention_error(got[l][b:b + 1], want) <= 2e-2
    one = torch.zeros(16, device=DEV)
    with pytest.raises(lpp.LppError) as e:
        lpp.lpp_tree_attention_layers(tree, lpp.LPP_BF16, lpp.LPP_F32, [], None, 1, 4, 4, 64, 64, 0.0, one)
    assert e.value.status == lpp.LPP_EINVAL
    with pytest.raises(lpp.LppError) as e:
        lpp.lpp_tree_attention_layers(tree, lpp.LPP_BF16, lpp.LPP_F32, [dict(q=one, k_cache=one, v_cache=one, k_tree=one,
                                                                             v_tree=None, out=one)],
                                      None, 1, 4, 4, 64, 64, 0.0, one)
    assert e.value.status == lpp.LPP_EINVAL


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("L,Hkv,seq", [(1, 2, [1100, 333]), (3, 4, None), (3, 1, [0, 1099]), (17, 2, None)])
@pytest.mark.parametrize("out_dtype", [lpp.LPP_F32, lpp.LPP_BF16])
def test_layers_float32_keys_in_ranges(Dh, L, Hkv, seq, out_dtype):
    # 1100 keys in two to four ranges (17 layers: two launches that share the partials): shared heads, ragged
    # lengths, bf16 output; 21 rows, so the second row tile is a short one
    cfg = CONFIGS[2].scaled(N=20, S=1100, H=4, B=2 if seq else 1, Dh=Dh, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N)
    atts = [_layer_inputs(cfg, Hkv, l) for l in range(L)]
    got = _run_layers(lpp.Tree(parent), atts, cfg, Hkv, out_dtype=out_dtype, seq_len=seq)
    tol = 1e-4 if out_dtype == lpp.LPP_F32 else 2.0 ** -8       # (half a unit of bf16's last place)
    for l in range(L):
        for b in range(cfg.B):
            n = seq[b] if seq else cfg.S
            want = tree_attention(atts[l]["q"][b:b + 1], atts[l]["kc"][b:b + 1, :, :n], atts[l]["vc"][b:b + 1, :, :n],
                                  atts[l]["kt"][b:b + 1], atts[l]["vt"][b:b + 1], parent)
            assert attention_error(got[l][b:b + 1], want) <= tol, (l, b)


@pytest.mark.parametrize("Dh", [64, 128])
def test_float32_takes_fewer_ranges_for_a_smaller_workspace(Dh):
    # every size that is accepted gives the result and leaves what lies behind it alone
    cfg = CONFIGS[2].scaled(N=20, S=4000, H=4, B=1, Dh=Dh, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    att = _layer_inputs(cfg, cfg.H, 0)
    want = tree_attention(att["q"], att["kc"], att["vc"], att["kt"], att["vt"], parent)
    t = {n: dev(att[n]) for n in ("q", "kc", "vc", "kt", "vt")}
    full = lpp.lpp_tree_attention_workspace(tree, 1, cfg.H, cfg.S, Dh)
    least = 0
    for part in range(1, 33):
        size = full * part // 32 // 16 * 16
        ws = torch.full((full + 256,), 0x5A, dtype=torch.uint8, device=DEV)
        out = torch.full((1, cfg.H, cfg.M, Dh), float("nan"), device=DEV)
        try:
            lpp.lpp_tree_attention(tree, lpp.LPP_F32, t["q"], t["kc"], t["vc"], t["kt"], t["vt"], None, 1, cfg.H, cfg.S,
                                   Dh, 0.0, out, ws[:size])
        except lpp.LppError as e:
            assert e.status == lpp.LPP_ENOWORKSPACE and least == 0
            continue
        least = least or part
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5A).all())
        assert attention_error(out.cpu().numpy(), want) <= 1e-4, part
    assert 1 <= least < 32


def test_float32_needs_room_for_one_range_only():
    # of 16 that the query's size has room for, whatever bf16 would ask for at these sizes (8)
    cfg = CONFIGS[2].scaled(N=20, S=4000, H=4, B=1, kv_dtype="f32")
    parent = static_tree(cfg.branching, cfg.N)
    att = _layer_inputs(cfg, cfg.H, 0)
    t = {n: dev(att[n]) for n in ("q", "kc", "vc", "kt", "vt")}
    ws = torch.empty(cfg.H * 32 * (cfg.Dh + 2) * 4 + 256, dtype=torch.uint8, device=DEV)
    out = torch.full((1, cfg.H, cfg.M, cfg.Dh), float("nan"), device=DEV)
    tree = lpp.Tree(parent)
    lpp.lpp_tree_attention(tree, lpp.LPP_F32, t["q"], t["kc"], t["vc"], t["kt"], t["vt"], None, 1, cfg.H, cfg.S, cfg.Dh, 0.0, out, ws)
    want = tree_attention(att["q"], att["kc"], att["vc"], att["kt"], att["vt"], parent)
    assert attention_error(out.cpu().numpy(), want) <= 1e-4


@pytest.mark.parametrize("N,S,B,H,Hkv,Dh,L,ragged", [
    (45, 100, 12, 24, 24, 64, 1, False),     # 288 heads, seven key groups
    (60, 70, 8, 30, 10, 64, 1, True),        # four
    (45, 1100, 12, 24, 8, 64, 1, True),      # all rows of a head in one block
    (60, 1100, 3, 31, 31, 64, 3, False),     # padding behind each layer's last heads
    (20, 2600, 11, 30, 30, 128, 1, True),    # long rows
    (60, 3000, 5, 20, 20, 64, 1, True),      # 200 blocks of 8 waves
    (128, 50, 6, 24, 24, 64, 1, True),       # 129 rows: five tiles and four
    (128, 1100, 11, 12, 4, 64, 1, False),    # the same, long caches
    (12, 70, 12, 24, 24, 64, 1, True), (12, 70, 12, 24, 8, 128, 1, True),      # one tile, blocks of 4 waves
    (60, 120, 5, 28, 28, 128, 1, True),      # long rows, blocks of 4 waves
])
def test_layers_launch_shapes(N, S, B, H, Hkv, Dh, L, ragged):
    branching = (6, 3, 2, 2, 1, 1) if N <= 60 else (8, 4, 2, 2, 1, 1, 1, 1)
    cfg = CONFIGS[2].scaled(N=N, branching=branching, S=S, H=H, B=B, Dh=Dh)
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    atts = [_layer_inputs(cfg, Hkv, l) for l in range(L)]
    seq = [(S * (b + 1) // B if b != 1 else 0) for b in range(B)] if ragged else [S] * B
    got = _run_layers(tree, atts, cfg, Hkv, seq_len=seq if ragged else None)
    again = _run_layers(tree, atts, cfg, Hkv, seq_len=seq if ragged else None)
    gq = H // Hkv
    for l in range(L):
        assert np.all(np.isfinite(got[l])) and np.array_equal(got[l], again[l])
        for b in range(B):
            for h in {(7 * b + l) % H, (H - 1 - b) % H}:
                k = slice(h // gq, h // gq + 1)
                want = tree_attention(atts[l]["q"][b:b + 1, h:h + 1], atts[l]["kc"][b:b + 1, k, :seq[b]],
                                      atts[l]["vc"][b:b + 1, k, :seq[b]], atts[l]["kt"][b:b + 1, k], atts[l]["vt"][b:b + 1, k], parent)
                assert attention_error(got[l][b:b + 1, h:h + 1], want) <= TOL["bf16"], (l, b, h)


@pytest.mark.parametrize("N,S,B,H,sizes", [(45, 1100, 12, 24, 1), (60, 3000, 5, 20, 1), (26, 1024, 1, 16, 9), (20, 2481, 1, 16, 9), (10, 4075, 1, 20, 6)])
def test_bf16_shares_no_range_for_a_smaller_workspace(N, S, B, H, sizes):
    # half of what is asked for where two blocks share a range, no less (the last: what the float32 call asks for is more): every size that is accepted gives the result, the order of
    # the float32 sums over waves apart, and leaves what lies behind it alone
    cfg = CONFIGS[2].scaled(N=N, branching=(6, 3, 2, 2, 1, 1), S=S, H=H, B=B)
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    att = _layer_inputs(cfg, H, 0)
    t = {n: bf16_dev(att[n + "_bits"]) for n in ("q", "kc", "vc", "kt", "vt")}
    full = lpp.lpp_tree_attention_workspace(tree, B, H, S, cfg.Dh)
    outs = []
    for part in range(1, 17):
        size = full * part // 16 // 256 * 256
        ws = torch.full((full + 256,), 0x5A, dtype=torch.uint8, device=DEV)
        out = torch.full((B, H, cfg.M, cfg.Dh), float("nan"), device=DEV)
        try:
            lpp.lpp_tree_attention(tree, lpp.LPP_BF16, t["q"], t["kc"], t["vc"], t["kt"], t["vt"], None, B, H, S, cfg.Dh, 0.0, out,
                                   ws[:size])
        except lpp.LppError as e:
            assert e.status == lpp.LPP_ENOWORKSPACE and not outs
            continue
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5A).all())
        outs.append(out.cpu().numpy())
    assert len(outs) == sizes
    want = tree_attention(att["q"][-1:, -1:], att["kc"][-1:, -1:], att["vc"][-1:, -1:], att["kt"][-1:, -1:], att["vt"][-1:, -1:], parent)
    assert max(attention_error(o[-1:, -1:], want) for o in outs) <= TOL["bf16"]
    assert max(attention_error(o, outs[-1]) for o in outs) <= 2e-6


@pytest.mark.parametrize("N,S,B,H,Dh", [(30, 3000, 12, 24, 64), (45, 1100, 12, 24, 64), (128, 1100, 11, 12, 64), (20, 2600, 11, 30, 128), (60, 3000, 5, 20, 64)])
def test_launches_of_many_blocks_leave_workspace_and_handle_alone(N, S, B, H, Dh):
    # no partial results, and so no tickets in the tree handle: such a call has nothing that another on the same handle could take
    cfg = CONFIGS[2].scaled(N=N, branching=(8, 4, 2, 2, 1, 1, 1, 1), S=S, H=H, B=B, Dh=Dh)
    tree = lpp.Tree(static_tree(cfg.branching, cfg.N))

    def zeros(rows):
        return torch.zeros(B, H, rows, Dh, dtype=torch.bfloat16, device=DEV)

    ws = torch.full((lpp.lpp_tree_attention_workspace(tree, B, H, S, Dh),), 0x5A, dtype=torch.uint8, device=DEV)
    out = torch.empty(B, H, cfg.M, Dh, device=DEV)
    lpp.lpp_tree_attention(tree, lpp.LPP_BF16, zeros(cfg.M), zeros(S), zeros(S), zeros(cfg.M), zeros(cfg.M), None, B, H, S, Dh, 0.0, out, ws)
    assert bool((ws == 0x5A).all()) and bool((out == 0).all())


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("B,H,Hkv,N,S,L", [
    (1, 1, 1, 8, 4000, 1), (1, 2, 1, 15, 64, 1), (1, 3, 3, 16, 700, 2), (1, 4, 1, 99, 130, 1), (1, 5, 5, 20, 1500, 1), (1, 6, 2, 31, 33, 3),
    (1, 7, 7, 60, 900, 1), (1, 9, 9, 26, 1024, 1), (3, 4, 2, 45, 500, 1), (1, 12, 6, 100, 300, 2), (2, 20, 20, 9, 800, 1), (5, 8, 4, 61, 0, 1),
    (3, 16, 16, 43, 1200, 1), (1, 33, 11, 17, 31, 1)])
def test_launches_of_few_blocks(Dh, B, H, Hkv, N, S, L):
    # 1 to 96 heads: key/value heads that are no multiple of 8, alone and behind eights of them, one and two tiles a wave, blocks
    # of 4 and 8 waves, up to 15 key ranges and none, ragged lengths with items that leave waves and whole ranges empty
    cfg = CONFIGS[2].scaled(N=N, S=S, H=H, B=B, Dh=Dh, branching=(8, 4, 2, 2, 1, 1, 1, 1))
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    atts = [_layer_inputs(cfg, Hkv, l) for l in range(L)]
    for seq in (None, [S - b * S // B if b else S // 3 for b in range(B)]):
        got = _run_layers(tree, atts, cfg, Hkv, seq_len=seq)
        again = _run_layers(tree, atts, cfg, Hkv, seq_len=seq)
        for l in range(L):
            assert np.array_equal(got[l], again[l])
            for b in range(B):
                n = S if seq is None else seq[b]
                want = tree_attention(atts[l]["q"][b:b + 1], atts[l]["kc"][b:b + 1, :, :n], atts[l]["vc"][b:b + 1, :, :n],
                                      atts[l]["kt"][b:b + 1], atts[l]["vt"][b:b + 1], parent)
                assert attention_error(got[l][b:b + 1], want) <= TOL["bf16"]


@pytest.mark.parametrize("B,H,Hkv", [(65, 256, 256), (1041, 20, 4)])
def test_layers_of_many_units_are_those_of_single_calls(B, H, Hkv):
    # 16640 and 20820 heads a layer: more than a launch of 16 layers can tell apart by reciprocals
    tree = lpp.Tree(np.asarray([-1, 0, 0, 1], dtype=np.int32))
    M, S, Dh, L = 4, 16, 64, 17
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)

    def normal(heads, rows):
        return torch.randn(B, heads, rows, Dh, generator=gen, device=DEV).to(torch.bfloat16)

    layers = [dict(q=normal(H, M), k_cache=normal(Hkv, S), v_cache=normal(Hkv, S), k_tree=normal(Hkv, M), v_tree=normal(Hkv, M),
                   out=torch.full((B, H, M, Dh), float("nan"), device=DEV)) for _ in range(L)]
    ws = torch.empty(lpp.lpp_tree_attention_layers_workspace(tree, L, B, H, S, Dh), dtype=torch.uint8, device=DEV)
    lpp.lpp_tree_attention_layers(tree, lpp.LPP_BF16, lpp.LPP_F32, layers, None, B, H, Hkv, S, Dh, 0.0, ws)
    one = torch.empty(B, H, M, Dh, device=DEV)
    for y in layers:
        lpp.lpp_tree_attention_layers(tree, lpp.LPP_BF16, lpp.LPP_F32, [dict(y, out=one)], None, B, H, Hkv, S, Dh, 0.0, ws)
        assert torch.equal(y["out"], one)
