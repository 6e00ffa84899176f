"""What this library's speed is judged by: one pass of each of its public calls, at the sizes its users run them.

The sizes are the five shapes of ``workloads/configs.py`` (the verification step of visual auto-regressive
models: LlamaGen-like 16384-code codebooks of dimension 8, a Lumina-like image slice of 8192 codes of
dimension 256 inside a 65536-wide logit row) with the options the header offers: ragged caches, shared
key/value heads, several layers per call, guidance and top-k in front of the target, distinct siblings.
``draw`` spreads the same parameters over the range between the smallest and the largest of them.

A case has a ``path``:
  neighbours  the neighbour table of a codebook, once per codebook
  attention   tree-masked attention of one layer, or of several layers in one call
  verify      softmax, relaxed acceptance and walk of a whole batch
  step        one decode step of a one-layer target: attention, verify, commit to the cache
"""
import math

import numpy as np
import torch

import paper_2502_06352_amd as lpp

TREE_S, TREE_L, TREE_XXL, TREE_WIDE = "4,2,1,1", "4,2,2,1,1", "6,3,2,2,1,1", "8,4,2,2,1,1,1,1"
MOST_KV = 16 * 24 * 4096 * 64            # cached elements of K (and of V) in the largest case
MOST_PAIRS = 8192 * 8192 * 256           # V * V * D of the largest codebook (D as a power of two)


# ------------------------------------------------------------------------------------------ cases

def _attention(name, **kw):
    c = dict(name=name, path="attention", B=1, H=16, Hkv=16, Dh=64, S=1024, N=26, tree=TREE_L, dtype="bf16", out="f32",
             layers=1, ragged=False)
    c.update(kw)
    return c


def _verify(name, **kw):
    c = dict(name=name, path="verify", B=1, V=16384, ldv=16384, offset=0, D=8, k=1000, bound=3.0, sigma=2.0, N=60,
             tree=TREE_XXL, guidance=0.0, top_k=0, rule="prefix", siblings="iid")
    c.update(kw)
    return c


def _step(name, **kw):
    c = _verify(name, B=1)
    c.update(_attention(name, path="step", ragged=True))
    c.update(kw)
    return c


def listed():
    return [
        # the table of a small codebook: launches and latency
        dict(name="neighbours_small", path="neighbours", V=1024, D=8, k=16),
        # the table of a LlamaGen-like codebook, at the neighbourhood size the method is run with
        dict(name="neighbours_d8", path="neighbours", V=16384, D=8, k=1000),
        # the table of a Chameleon / Lumina-like codebook: long rows, the dense contraction
        dict(name="neighbours_d256", path="neighbours", V=8192, D=256, k=1000),
        # float32 attention of a small model: the smallest call
        _attention("attention_f32_small", H=4, Hkv=4, S=256, N=15, tree=TREE_S, dtype="f32"),
        # one layer of a Lumina-like target at batch 1 with shared key/value heads and bf16 activations
        _attention("attention_gqa_b1", H=32, Hkv=8, Dh=128, S=2400, N=60, tree=TREE_XXL, out="bf16"),
        # the layers of a LlamaGen-XXL-like target in one call, the batch's items at different positions of the image
        _attention("attention_16_layers", B=4, H=24, Hkv=24, N=60, tree=TREE_XXL, out="bf16", layers=16, ragged=True),
        # a large batch of long images with a wide tree
        _attention("attention_large", B=16, H=24, Hkv=24, S=4096, N=128, tree=TREE_WIDE),
        # batch 1 with the sampling configuration of the experiments: guidance 3, top-k 2000
        _verify("verify_guided_b1", V=8192, ldv=65536, offset=4, D=256, bound=2.0, guidance=3.0, top_k=2000),
        # the batched step with distinct siblings
        _verify("verify_distinct", B=4, siblings="distinct"),
        # a large batch with a wide tree
        _verify("verify_large", B=16, N=128, tree=TREE_WIDE),
        # a whole step at batch 1: latency
        _step("step_b1", bound=2.0, k=100),
        # a whole step of the headline shape
        _step("step_b4", B=4, H=24, Hkv=24, N=60, tree=TREE_XXL),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_tree(rng, c):
    c["N"] = _log_int(rng, 8, 128)
    c["tree"] = TREE_L if c["N"] <= 40 else rng.choice((TREE_XXL, TREE_WIDE))


def _kv_elements(c):
    return c["B"] * c["H"] * (c["S"] + 3 * c["N"]) * c["Dh"]


def _draw_attention(rng, c, most):
    c["H"] = rng.choice((4, 8, 12, 16, 20, 24, 32))
    c["Hkv"] = c["H"] // rng.choice((1, 1, 2, 4))
    c["Dh"] = rng.choice((64, 64, 128))
    c["S"] = _log_int(rng, 64, 4096)
    c["B"] = _log_int(rng, 1, max(1, min(16, most // _kv_elements(dict(c, B=1)))))
    c["out"] = rng.choice(("f32", "bf16"))
    c["ragged"] = rng.random() < 0.5


def _draw_verify(rng, c):
    c["V"] = _log_int(rng, 1024, 16384)
    if rng.random() < 0.6:
        c["V"] -= c["V"] % 4                        # rows that start on 16 bytes
    c["offset"] = rng.choice((0, 0, 4))
    c["ldv"] = c["V"] + c["offset"]
    c["D"] = 8
    c["k"] = _log_int(rng, 16, min(1000, c["V"]))
    c["bound"] = rng.choice((2.0, 3.0))
    c["sigma"] = rng.uniform(1.5, 2.0)


def draw(rng):
    path = rng.choice(("neighbours", "attention", "attention", "verify", "verify", "step"))
    if path == "neighbours":
        D = _log_int(rng, 4, 256)
        pad = 1 << max(4, (D - 1).bit_length())
        V = _log_int(rng, 256, min(16384, int(math.sqrt(MOST_PAIRS / pad))))
        return dict(path=path, V=V, D=D, k=_log_int(rng, 8, min(1000, V)))
    if path == "attention":
        c = _attention("")
        c["dtype"] = "f32" if rng.random() < 0.2 else "bf16"
        most = MOST_KV // (32 if c["dtype"] == "f32" else 1)
        _draw_tree(rng, c)
        _draw_attention(rng, c, most)
        c["layers"] = _log_int(rng, 1, max(1, min(32, most // _kv_elements(c)))) if rng.random() < 0.5 else 1
    elif path == "verify":
        c = _verify("", B=_log_int(rng, 1, 16))
        _draw_verify(rng, c)
        _draw_tree(rng, c)
        if rng.random() < 0.4:
            c["guidance"], c["top_k"] = rng.choice((0.0, 3.0)), min(2000, c["V"] // 2)
        c["siblings"] = rng.choice(("iid", "iid", "distinct"))
        c["rule"] = "skip" if rng.random() < 0.15 else "prefix"
    else:
        c = _step("")
        _draw_tree(rng, c)
        _draw_attention(rng, c, MOST_KV // 4)
        c["ragged"] = True
        _draw_verify(rng, c)
    del c["name"]
    return c


# ----------------------------------------------------------------------------------------- inputs

def _tree(c):
    """Left-heavy static tree: of the full tree with the given branching, the N nodes with the least sum of
    depth x rank, numbered by depth."""
    branching = [int(x) for x in c["tree"].split(",")]
    level, nodes = [()], []
    for b in branching:
        level = [p + (r,) for p in level for r in range(b)]
        nodes += level
    nodes.sort(key=lambda p: (sum((i + 1) * r for i, r in enumerate(p)), len(p), p))
    kept = sorted(nodes[:c["N"]], key=lambda p: (len(p), p))
    row = {p: i + 1 for i, p in enumerate(kept)}
    row[()] = 0
    return [-1] + [row[p[:-1]] for p in kept]


def _depth(parent):
    d = [0]
    for p in parent[1:]:
        d.append(d[p] + 1)
    return max(max(d), 1)


def _seq_lens(c, parent):
    """Valid cache length of every item: half way to full over the batch when ragged; a step leaves room for the
    rows it commits."""
    full = c["S"] - (_depth(parent) + 1 if c["path"] == "step" else 0)
    if not c["ragged"]:
        return [full] * c["B"]
    return [full - b * full // (2 * c["B"]) for b in range(c["B"])]


def _codebook(gen, V, D):
    e = torch.randn(V, D, generator=gen, device="cuda", dtype=torch.float64)
    return (e / e.norm(dim=1, keepdim=True)).float()


def _build(E, k, neigh, ws):
    lpp.lpp_build_neighbours(E, k, neigh, ws)
    return neigh


def _prepare_neighbours(V, D, k, gen):
    ws = torch.empty(lpp.lpp_build_neighbours_workspace(V, D, k), dtype=torch.uint8, device="cuda")
    return dict(E=_codebook(gen, V, D), k=k, neigh=torch.empty((V, k), dtype=torch.int32, device="cuda"), ws=ws)


def _prepare_attention(c, parent, tree, gen):
    B, H, Hkv, M, S, Dh, L = c["B"], c["H"], c["Hkv"], len(parent), c["S"], c["Dh"], c["layers"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    odt = torch.bfloat16 if c["out"] == "bf16" else torch.float32

    def normal(heads, rows):
        return torch.randn(B, heads, rows, Dh, generator=gen, device="cuda", dtype=torch.float32).to(dt)

    layers = [dict(q=normal(H, M), k_cache=normal(Hkv, S), v_cache=normal(Hkv, S), k_tree=normal(Hkv, M),
                   v_tree=normal(Hkv, M), out=torch.empty((B, H, M, Dh), dtype=odt, device="cuda")) for _ in range(L)]
    ws = lpp.lpp_tree_attention_layers_workspace(tree, L, B, H, S, Dh)
    seq = torch.tensor(_seq_lens(c, parent), dtype=torch.int32, device="cuda") if c["ragged"] else None
    return dict(layers=layers, seq_len=seq, attn_ws=torch.empty(max(ws, 256), dtype=torch.uint8, device="cuda"),
                dtype=lpp.LPP_BF16 if c["dtype"] == "bf16" else lpp.LPP_F32,
                out_dtype=lpp.LPP_BF16 if c["out"] == "bf16" else lpp.LPP_F32)


def _prepare_verify(c, parent, tree, gen):
    B, M, V, off, ldv = c["B"], len(parent), c["V"], c["offset"], c["ldv"]

    def rows():
        full = torch.full((B, M, ldv), -math.inf, device="cuda")
        return full, full[:, :, off:off + V]

    def normal():
        return torch.randn(B, M, V, generator=gen, device="cuda") * c["sigma"]

    # the drafter tracks the target: correlation 0.8, the same spread
    target, t = rows()
    t.copy_(normal())
    drafter, d = rows()
    d.copy_(0.8 * t + 0.6 * normal())
    uncond = None
    if c["guidance"]:
        uncond, u = rows()
        u.copy_(normal())
    kids = [[] for _ in range(M)]
    for i in range(1, M):
        kids[parent[i]].append(i)
    tokens = torch.zeros((B, M), dtype=torch.int32, device="cuda")
    most = max(len(x) for x in kids)
    for b in range(B):
        p = torch.softmax(d[b], dim=-1)
        drawn = torch.multinomial(p, most, replacement=c["siblings"] == "iid", generator=gen).int()
        for P in range(M):
            if kids[P]:
                tokens[b, kids[P][0]:kids[P][-1] + 1] = drawn[P, :len(kids[P])]      # children are consecutive rows
    n = _prepare_neighbours(V, c["D"], c["k"], gen)
    neigh = _build(n["E"], n["k"], n["neigh"], n["ws"])

    def out(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    i32 = torch.int32
    res = dict(accept_len=out(B, dtype=i32), path=out(B, max(tree.depth, 1), dtype=i32), final_token=out(B, dtype=i32),
               decision=out(B, M, dtype=torch.uint8), ratio=out(B, M), mass=out(B, M), n_agg=out(B, M, dtype=i32),
               q_tok=out(B, M), p_tok=out(B, M), final_tok_all=out(B, M, dtype=i32))
    ws = torch.empty(lpp.lpp_relaxed_verify_workspace(tree, B, V, c["k"]), dtype=torch.uint8, device="cuda")
    return dict(target=target, uncond=uncond, drafter=drafter, tokens=tokens, neigh=neigh, verify_out=res, verify_ws=ws,
                u_accept=torch.rand(B, M, generator=gen, device="cuda"),
                u_final=torch.rand(B, M, generator=gen, device="cuda"))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    c = dict(case)
    if c["path"] == "neighbours":
        return dict(case=c, **_prepare_neighbours(c["V"], c["D"], c["k"], gen))
    parent = _tree(c)
    tree = lpp.Tree(np.asarray(parent, dtype=np.int32))
    state = dict(case=c, tree=tree)
    if c["path"] in ("attention", "step"):
        state.update(_prepare_attention(c, parent, tree, gen))
    if c["path"] in ("verify", "step"):
        state.update(_prepare_verify(c, parent, tree, gen))
    if c["path"] == "step":
        state["new_len"] = torch.empty(c["B"], dtype=torch.int32, device="cuda")
    return state


# ------------------------------------------------------------------------------------------- pass

def _run_attention(s):
    c, tree = s["case"], s["tree"]
    B, H, Hkv, S, Dh = c["B"], c["H"], c["Hkv"], c["S"], c["Dh"]
    y = s["layers"][0]
    if len(s["layers"]) > 1:
        lpp.lpp_tree_attention_layers(tree, s["dtype"], s["out_dtype"], s["layers"], s["seq_len"], B, H, Hkv, S, Dh, 0.0,
                                      s["attn_ws"])
    elif Hkv != H or c["out"] == "bf16":
        lpp.lpp_tree_attention_gqa(tree, s["dtype"], s["out_dtype"], y["q"], y["k_cache"], y["v_cache"], y["k_tree"],
                                   y["v_tree"], s["seq_len"], B, H, Hkv, S, Dh, 0.0, y["out"], s["attn_ws"])
    else:
        lpp.lpp_tree_attention(tree, s["dtype"], y["q"], y["k_cache"], y["v_cache"], y["k_tree"], y["v_tree"],
                               s["seq_len"], B, H, S, Dh, 0.0, y["out"], s["attn_ws"])
    return [x["out"] for x in s["layers"]]


def _run_verify(s):
    c = s["case"]
    rows = (c["ldv"], c["offset"], c["V"], c["B"], s["tokens"], s["neigh"], c["k"], c["k"])
    draws = (s["u_accept"], s["u_final"], s["verify_out"], s["verify_ws"])
    if c["rule"] == "skip" or c["siblings"] == "distinct":
        lpp.lpp_relaxed_verify_opts(
            s["tree"], s["target"], s["drafter"], *rows, *draws, bound=lpp.LPP_BOUND_MULTIPLICATIVE,
            bound_value=c["bound"], rule=lpp.LPP_RULE_SKIP if c["rule"] == "skip" else lpp.LPP_RULE_PREFIX,
            siblings=lpp.LPP_SIBLINGS_DISTINCT if c["siblings"] == "distinct" else lpp.LPP_SIBLINGS_IID,
            uncond_logits=s["uncond"], cfg_scale=c["guidance"], top_k=c["top_k"])
    elif c["guidance"] or c["top_k"]:
        lpp.lpp_relaxed_verify_sampled(s["tree"], s["target"], s["uncond"], c["guidance"], c["top_k"], s["drafter"],
                                       *rows, c["bound"], *draws)
    else:
        lpp.lpp_relaxed_verify(s["tree"], s["target"], s["drafter"], *rows, c["bound"], *draws)
    return s["verify_out"]


def run(state):
    s = state
    path = s["case"]["path"]
    if path == "neighbours":
        return _build(s["E"], s["k"], s["neigh"], s["ws"])
    if path == "attention":
        return _run_attention(s)
    if path == "verify":
        return _run_verify(s)
    c, y, v = s["case"], s["layers"][0], s["verify_out"]
    _run_attention(s)
    _run_verify(s)
    lpp.lpp_commit_kv(s["tree"], s["dtype"], y["k_tree"], y["v_tree"], v["path"], v["accept_len"], s["seq_len"], c["B"],
                      c["Hkv"], c["S"], c["Dh"], y["k_cache"], y["v_cache"], s["new_len"])
    return dict(v, attention=y["out"], k_cache=y["k_cache"], v_cache=y["v_cache"], new_len=s["new_len"])


# -------------------------------------------------------------------------------- work, tolerance

def work(case):
    c = case
    if c["path"] == "neighbours":
        return {"bytes": 4 * c["V"] * (c["D"] + c["k"]), "flops": 2 * c["V"] * c["V"] * c["D"]}
    parent = _tree(c)
    B, M = c["B"], len(parent)
    nbytes = flops = 0
    if c["path"] in ("attention", "step"):
        e, eo = (2 if c["dtype"] == "bf16" else 4), (2 if c["out"] == "bf16" else 4)
        keys = sum(_seq_lens(c, parent))
        nbytes += c["layers"] * c["Dh"] * (2 * c["Hkv"] * keys * e + B * M * ((c["H"] + 2 * c["Hkv"]) * e + c["H"] * eo))
        flops += c["layers"] * 4 * c["H"] * M * (keys + B * M) * c["Dh"]
    if c["path"] in ("verify", "step"):
        # every row's target logits, the parents' drafter logits, the drafted tokens' neighbour lists
        logit_rows = M * (2 if c["guidance"] else 1) + len(set(parent) - {-1})
        nbytes += 4 * B * (c["V"] * logit_rows + c["N"] * c["k"])
        flops += 4 * B * c["V"] * logit_rows
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    c = case
    if c["path"] == "neighbours":
        return "exact"                              # indices; ties are settled by the definition
    # decisions, draws and set sizes are whole numbers that float32 sums settle: a tie now and then
    tol = {"rel": 2e-5, "differ": 0.005}
    if c["path"] in ("attention", "step"):
        tol["rel"] = 5e-3 if c["dtype"] == "bf16" or c["out"] == "bf16" else 1e-5
    return tol
