"""Helpers of the GPU parity tests: upload seeded inputs, call the C ABI through
the binding, bring results back, compare with the oracle under the stated rules."""
import numpy as np
import torch

import paper_2502_06352_amd as lpp
from oracle import build_neighbours, float32_error_bound, relaxed_verify
from workloads import children_lists

DEV = "cuda:0"


def dev(x, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(x))
    if dtype is not None:
        t = t.to(dtype)
    return t.to(DEV)


def bf16_dev(bits):
    """uint16 bit patterns -> torch.bfloat16 tensor on the device."""
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(DEV).view(torch.bfloat16)


def sparse_neighbour_table(E, k, tokens, V):
    """Oracle neighbour rows for the drafted tokens only; other rows hold a valid
    but arbitrary list (x, x+1, ...) that no node of this input reads."""
    neigh = ((np.arange(V, dtype=np.int64)[:, None] + np.arange(k, dtype=np.int64)[None, :]) % V).astype(np.int32)
    used = np.unique(tokens)
    neigh[used] = build_neighbours(E, k, rows=used)
    return neigh


def run_verify(tree, x, neigh, cfgV, off, ldv, k, lam, want_all=True, stream=None, additive=False, opts=None):
    """``opts``: None = the plain entry points; a dict (rule=, siblings=) = lpp_relaxed_verify_opts."""
    B, M = x["tokens"].shape
    depth = max(tree.depth, 1)
    d = {n: dev(x[n]) for n in ("target_logits", "drafter_logits", "tokens", "u_accept", "u_final")}
    dn = dev(neigh)
    out = {"accept_len": torch.full((B,), -7, dtype=torch.int32, device=DEV),
           "path": torch.full((B, depth), -7, dtype=torch.int32, device=DEV),
           "final_token": torch.full((B,), -7, dtype=torch.int32, device=DEV)}
    if want_all:
        out.update(decision=torch.full((B, M), 9, dtype=torch.uint8, device=DEV),
                   ratio=torch.zeros((B, M), device=DEV), mass=torch.zeros((B, M), device=DEV),
                   n_agg=torch.zeros((B, M), dtype=torch.int32, device=DEV),
                   q_tok=torch.zeros((B, M), device=DEV), p_tok=torch.zeros((B, M), device=DEV),
                   final_tok_all=torch.full((B, M), -7, dtype=torch.int32, device=DEV))
    ws = torch.empty(lpp.lpp_relaxed_verify_workspace(tree, B, cfgV, k), dtype=torch.uint8, device=DEV)
    if opts is not None:
        lpp.lpp_relaxed_verify_opts(tree, d["target_logits"], d["drafter_logits"], ldv, off, cfgV, B, d["tokens"], dn,
                                    neigh.shape[1], k, d["u_accept"], d["u_final"], out, ws, stream,
                                    bound=lpp.LPP_BOUND_ADDITIVE if additive else lpp.LPP_BOUND_MULTIPLICATIVE,
                                    bound_value=lam, **opts)
    else:
        call = lpp.lpp_relaxed_verify_additive if additive else lpp.lpp_relaxed_verify
        call(tree, d["target_logits"], d["drafter_logits"], ldv, off, cfgV, B, d["tokens"], dn,
             neigh.shape[1], k, lam, d["u_accept"], d["u_final"], out, ws, stream)
    torch.cuda.synchronize()
    return {n: t.cpu().numpy() for n, t in out.items()}


# Largest float32-cancellation allowance a node may be given (relative to the oracle's value): the
# oracle's bound can never hide an error larger than this, whatever it computes.
SLACK_CAP_REL = 1e-2


def compare_verify(parent, x, neigh, V, off, k, lam, got, rel=1e-4, tie=1e-5, cdf_tol=2e-6, additive=False,
                   rule="prefix", siblings="with_replacement", max_slack_used=None):
    """Compare every output with the float64 oracle.  Returns a report dict.

    Rules: decisions bit-exact unless |u - ratio| < tie (counted); mass / ratio / q_tok / p_tok
    within rel.  A value outside rel is still taken if it lies within rel plus the oracle's
    first-order bound on what float32 loses where Eq. 2's subtraction cancels
    (``float32_error_bound``, capped at SLACK_CAP_REL of the value): such values are counted in
    ``slack_used`` (at most ``max_slack_used`` of them, default 1 + nodes // 2000), and the report
    shows the true largest relative error (``max_rel``) and the largest allowance that was
    needed relative to the value (``max_slack_rel``).  n_agg equal unless the oracle's bound
    margin shows a float32-level tie at the stopping sum (counted); after such a tie the later
    siblings and the parent's draw are not comparable and are skipped (counted); final tokens
    must bracket u*Z in the oracle's float64 CDF within cdf_tol*Z.
    Under rule="skip" a tie can change more than one later membership, so the sizes may then
    differ by more than one.
    """
    want = relaxed_verify(parent, x["target_logits"], x["drafter_logits"], off, V, x["tokens"], neigh, k, lam,
                          x["u_accept"], x["u_final"], keep_final_cdf=True,
                          bound="additive" if additive else "multiplicative", rule=rule, siblings=siblings)
    ferr = None        # the float32 allowance: only worked out if some value falls outside rel
    kids = children_lists(parent)
    B, M = x["tokens"].shape
    rep = dict(nodes=0, near_tie_decisions=0, nagg_ties=0, skipped_after_tie=0, final_exact=0, final_rows=0,
               max_rel=0.0, slack_used=0, max_slack_rel=0.0, walks_compared=0)
    for b in range(B):
        tainted_rows = set()
        decision_uncertain = False
        for P in range(M):
            row_tainted = False
            for c in kids[P]:
                if row_tainted:
                    rep["skipped_after_tie"] += 1
                    decision_uncertain = True
                    continue
                rep["nodes"] += 1
                if got["n_agg"][b, c] != want["n_agg"][b, c]:
                    assert want["bound_margin"][b, c] < 1e-4, (
                        f"n_agg differs without a tie: b={b} c={c} got {got['n_agg'][b, c]} "
                        f"want {want['n_agg'][b, c]} margin {want['bound_margin'][b, c]}")
                    assert rule == "skip" or abs(int(got["n_agg"][b, c]) - int(want["n_agg"][b, c])) == 1
                    rep["nagg_ties"] += 1
                    row_tainted = True
                    decision_uncertain = True
                    continue
                if (rule == "skip" and want["bound_margin"][b, c] < 1e-6 and
                        abs(float(got["mass"][b, c]) - float(want["mass"][b, c])) > rel * abs(float(want["mass"][b, c]))):
                    # a neighbour whose sum meets the cap to within float32's rounding of the probabilities (2**-20):
                    # on the other side of the tie a later neighbour takes its place, as many in all
                    rep["nagg_ties"] += 1
                    row_tainted = True
                    decision_uncertain = True
                    continue
                for name in ("mass", "q_tok", "p_tok", "ratio"):
                    g, w = float(got[name][b, c]), float(want[name][b, c])
                    if g == w or (np.isnan(g) and np.isnan(w)):     # also +inf (p = 0) and 0/0 (p = 0 and no mass)
                        continue
                    err = abs(g - w) / max(abs(w), 1e-300)
                    rep["max_rel"] = max(rep["max_rel"], err)
                    if err <= rel:
                        continue
                    # outside the relative rule: what float32 can lose where Eq. 2's subtraction
                    # nearly cancels (the oracle's own bound, capped)
                    if ferr is None:
                        ferr = float32_error_bound(parent, x["target_logits"], x["drafter_logits"], off, V,
                                                   x["tokens"], neigh, k, lam,
                                                   bound="additive" if additive else "multiplicative", rule=rule,
                                                   siblings=siblings)
                    pt = max(float(want["p_tok"][b, c]), 1e-300)
                    slack = {"mass": ferr["mass_err"][b, c], "q_tok": ferr["q_tok_err"][b, c],
                             "p_tok": ferr["p_tok_err"][b, c],
                             "ratio": ferr["mass_err"][b, c] / pt + abs(w) * ferr["p_tok_err"][b, c] / pt}[name]
                    slack = min(float(slack), SLACK_CAP_REL * abs(w))
                    assert abs(g - w) <= rel * abs(w) + slack, (
                        f"{name} b={b} c={c}: got {g} want {w} rel {err} float32 allowance {slack}")
                    rep["slack_used"] += 1
                    rep["max_slack_rel"] = max(rep["max_slack_rel"], (abs(g - w) - rel * abs(w)) / max(abs(w), 1e-300))
                if got["decision"][b, c] != want["decision"][b, c]:
                    u = float(x["u_accept"][b, c])
                    assert abs(u - want["ratio"][b, c]) < tie, (
                        f"decision differs away from a tie: b={b} c={c} u={u} ratio={want['ratio'][b, c]}")
                    rep["near_tie_decisions"] += 1
                    decision_uncertain = True
            if row_tainted:
                tainted_rows.add(P)
                continue
            rep["final_rows"] += 1
            xg = int(got["final_tok_all"][b, P])
            assert 0 <= xg < V
            cdf = want["final_cdf"][b, P]
            Z = cdf[-1]
            tgt = float(x["u_final"][b, P]) * Z
            lo = cdf[xg - 1] if xg > 0 else 0.0
            assert lo - cdf_tol * Z <= tgt <= cdf[xg] + cdf_tol * Z, (
                f"final token outside its CDF bracket: b={b} P={P} got {xg} want {want['final_tok_all'][b, P]}")
            assert cdf[xg] - lo > 0, "drew a zero-probability token"
            rep["final_exact"] += int(xg == want["final_tok_all"][b, P])
        # the walk must be the walk of the decisions the GPU itself reports
        cur, n, path = 0, 0, []
        while True:
            nxt = next((c for c in kids[cur] if got["decision"][b, c]), None)
            if nxt is None:
                break
            path.append(nxt); cur = nxt; n += 1
        assert got["accept_len"][b] == n
        assert got["path"][b].tolist() == path + [-1] * (got["path"].shape[1] - n)
        assert got["final_token"][b] == got["final_tok_all"][b, cur]
        if not decision_uncertain:
            rep["walks_compared"] += 1
            assert got["accept_len"][b] == want["accept_len"][b]
            assert np.array_equal(got["path"][b], want["path"][b])
        assert np.all(got["decision"][b, 0] == 0)
    limit = 1 + rep["nodes"] // 2000 if max_slack_used is None else max_slack_used
    assert rep["slack_used"] <= limit, f"{rep['slack_used']} values needed the float32 allowance (limit {limit}): {rep}"
    return rep


def run_attention(tree, att, cfg, seq_len=None, S=None, stream=None):
    """Upload one attention input set and call lpp_tree_attention; returns float32 [B,H,M,Dh]."""
    B, H, M, Dh = att["q"].shape
    S = att["kc"].shape[2] if S is None else S
    if cfg.kv_dtype == "bf16":
        t = {n: bf16_dev(att[n + "_bits"]) for n in ("q", "kc", "vc", "kt", "vt")}
        dtype = lpp.LPP_BF16
    else:
        t = {n: dev(att[n]) for n in ("q", "kc", "vc", "kt", "vt")}
        dtype = lpp.LPP_F32
    sl = None if seq_len is None else dev(np.asarray(seq_len, dtype=np.int32))
    out = torch.full((B, H, M, Dh), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(max(lpp.lpp_tree_attention_workspace(tree, B, H, S, Dh), 256), dtype=torch.uint8, device=DEV)
    lpp.lpp_tree_attention(tree, dtype, t["q"], t["kc"] if S > 0 else None, t["vc"] if S > 0 else None,
                           t["kt"], t["vt"], sl, B, H, S, Dh, 0.0, out, ws, stream)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def attention_error(got, want):
    """max over rows of |got - want| / (|want| + max|want| over the row's Dh vector)."""
    scale = np.abs(want) + np.abs(want).max(axis=-1, keepdims=True)
    return float(np.max(np.abs(got - want) / scale))


def run_knn(E, k):
    V, D = E.shape
    dE = dev(E)
    neigh = torch.full((V, k), -1, dtype=torch.int32, device=DEV)
    nbytes = lpp.lpp_build_neighbours_workspace(V, D, k)
    assert nbytes > 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    lpp.lpp_build_neighbours(dE, k, neigh, ws)
    torch.cuda.synchronize()
    return neigh.cpu().numpy()
