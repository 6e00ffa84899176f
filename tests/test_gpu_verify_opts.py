"""GPU parity: lpp_relaxed_verify_opts (the other choice of A, distinct siblings, and their
combinations with both bounds) against the float64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import paper_2502_06352_amd as lpp
from workloads import CONFIGS, static_tree, make_codebook, make_verify_inputs
from gpu_common import run_verify, compare_verify, sparse_neighbour_table

pytestmark = pytest.mark.gpu


def _case(cfg, rho, skip=False, distinct=False, k=None, lam=None, additive=False, topk=0, salt=0, dup=False):
    parent = static_tree(cfg.branching, cfg.N)
    x = make_verify_inputs(cfg, parent, rho=rho, topk_filter=topk, salt=salt)
    if dup:                                     # a token handed in twice under one parent
        x["tokens"][:, 2] = x["tokens"][:, 1]
    E = make_codebook(cfg)
    k = cfg.k if k is None else k
    lam = cfg.lam if lam is None else lam
    neigh = sparse_neighbour_table(E, k, x["tokens"][:, 1:], cfg.V)
    tree = lpp.Tree(parent)
    opts = dict(rule=lpp.LPP_RULE_SKIP if skip else lpp.LPP_RULE_PREFIX,
                siblings=lpp.LPP_SIBLINGS_DISTINCT if distinct else lpp.LPP_SIBLINGS_IID)
    got = run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, k, lam, additive=additive, opts=opts)
    rep = compare_verify(parent, x, neigh, cfg.V, cfg.vocab_offset, k, lam, got, additive=additive,
                         rule="skip" if skip else "prefix",
                         siblings="without_replacement" if distinct else "with_replacement")
    print(f"cfg{cfg.idx} rho={rho} skip={skip} distinct={distinct} k={k} lam={lam}: {rep} "
          f"mean n_agg={got['n_agg'][:, 1:].mean():.1f} accept_len={got['accept_len'].mean():.2f}", flush=True)
    return rep, got, (tree, x, neigh, k, lam)


@pytest.mark.parametrize("idx", [1, 2, 3, 4])
@pytest.mark.parametrize("skip,distinct", [(True, False), (False, True), (True, True)])
def test_opts_parity_configs(idx, skip, distinct):
    rep, got, _ = _case(CONFIGS[idx], 0.8, skip=skip, distinct=distinct)
    assert rep["nodes"] > 0 and rep["near_tie_decisions"] <= 2
    assert rep["nagg_ties"] <= (6 if skip else 2)


def test_opts_defaults_equal_the_plain_entry_points():
    cfg = CONFIGS[3]
    rep, got, (tree, x, neigh, k, lam) = _case(cfg, 0.8)
    plain = run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, k, lam)
    for n in got:
        assert np.array_equal(got[n], plain[n]), n
    add = run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, k, 0.05, additive=True)
    add2 = run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, k, 0.05, additive=True,
                      opts=dict(rule=lpp.LPP_RULE_PREFIX, siblings=lpp.LPP_SIBLINGS_IID))
    for n in add:
        assert np.array_equal(add[n], add2[n]), n


def test_opts_skip_rule_differs_from_prefix_and_contains_it():
    cfg = CONFIGS[3]
    _, sk, (tree, x, neigh, k, lam) = _case(cfg, 0.8, skip=True)
    pre = run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, k, lam)
    assert np.all(sk["n_agg"] >= pre["n_agg"]) and np.any(sk["n_agg"] > pre["n_agg"])
    # first children see the same r under both rules: their mass can only grow (up to float32 rounding order)
    parent = static_tree(cfg.branching, cfg.N)
    first = [c for c in range(1, cfg.M) if c == 1 or parent[c] != parent[c - 1]]
    assert np.all(sk["mass"][:, first] >= pre["mass"][:, first] * (1 - 1e-5))


@pytest.mark.parametrize("additive,lam", [(False, 3.0), (True, 0.02)])
def test_opts_skip_rule_stress_full_batch_and_filtered_targets(additive, lam):
    rep, got, _ = _case(CONFIGS[5], 0.8, skip=True, distinct=True, additive=additive, lam=lam)
    assert rep["nodes"] + rep["skipped_after_tie"] == 16 * 128        # (nodes counts the tied ones too)
    rep, _, _ = _case(CONFIGS[3].scaled(B=2), 0.8, skip=True, additive=additive, lam=lam, topk=2000)
    assert rep["nodes"] > 0


@pytest.mark.parametrize("k,lam", [(1, 3.0), (1000, 1.0), (1000, 0.5), (7, 50.0), (1000, 1e9), (4096, 1.5)])
def test_opts_special_cases(k, lam):
    cfg = CONFIGS[3].scaled(B=1)
    _case(cfg, 0.8, skip=True, distinct=True, k=k, lam=lam)


def test_opts_distinct_siblings_repeated_token_and_ragged_vocab():
    rep, got, _ = _case(CONFIGS[2], 0.8, distinct=True, dup=True)
    assert got["p_tok"][0, 2] == 0.0                       # the second copy has no drafter mass left
    cfg = CONFIGS[2].scaled(V=5003, ldv=5100, vocab_offset=3, k=37, N=26)
    _case(cfg, 0.8, skip=True, distinct=True)
    cfg = CONFIGS[1].scaled(V=33, ldv=40, vocab_offset=1, k=33)
    _case(cfg, 0.5, skip=True, distinct=True, lam=4.0)


@pytest.mark.parametrize("skip,distinct", [(True, False), (False, True)])
@pytest.mark.parametrize("V,off", [(16384, 0), (8192, 4), (5003, 3), (3001, 0), (1027, 1), (20001, 3)])
def test_opts_more_rows_than_compute_units(V, off, skip, distinct):
    # 305 rows: the walk goes by tickets, in every width of the kernel
    rep, _, _ = _case(CONFIGS[3].scaled(V=V, ldv=V + off, vocab_offset=off, B=5, k=min(700, V // 2)), 0.8, skip=skip, distinct=distinct)
    assert rep["nodes"] > 0 and rep["near_tie_decisions"] <= 2
    assert rep["nagg_ties"] <= (rep["nodes"] // 100 + 2 if skip else 2)


@pytest.mark.parametrize("B", [1, 3, 4])                  # tickets, tickets, the resident grid: where one is the faster
@pytest.mark.parametrize("V", [20000, 32768])
def test_opts_distinct_siblings_of_wide_rows(V, B):
    rep, _, _ = _case(CONFIGS[3].scaled(V=V, ldv=V, B=B, k=300), 0.8, distinct=True)
    assert rep["nodes"] > 0 and rep["near_tie_decisions"] <= 2 and rep["nagg_ties"] <= 2


def test_opts_argument_errors():
    cfg = CONFIGS[1]
    parent = static_tree(cfg.branching, cfg.N)
    x = make_verify_inputs(cfg, parent, rho=0.5)
    neigh = sparse_neighbour_table(make_codebook(cfg), cfg.k, x["tokens"][:, 1:], cfg.V)
    tree = lpp.Tree(parent)
    for bad in (dict(rule=2), dict(siblings=-1), dict(rule=0, siblings=7)):
        with pytest.raises(lpp.LppError) as e:
            run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, cfg.k, cfg.lam, opts=bad)
        assert e.value.status == lpp.LPP_EINVAL


@pytest.mark.parametrize("additive,lam", [(False, 3.0), (True, 0.05)])
def test_opts_everything_at_once_front_end_skip_rule_distinct_siblings(additive, lam):
    """Guidance + top-k in front, the skip rule and distinct siblings behind, either bound: the oracle
    pipeline is sampling_frontend -> relaxed_verify with the same options."""
    from oracle import sampling_frontend
    from gpu_common import DEV, dev
    cfg = CONFIGS[3].scaled(B=2)
    parent = static_tree(cfg.branching, cfg.N)
    tree = lpp.Tree(parent)
    x = make_verify_inputs(cfg, parent, rho=0.8, salt=3)
    y = make_verify_inputs(cfg, parent, rho=0.0, salt=103)
    V, off, k = cfg.V, cfg.vocab_offset, cfg.k
    B, M = x["tokens"].shape
    neigh = sparse_neighbour_table(make_codebook(cfg), k, x["tokens"][:, 1:], V)
    out = {"accept_len": torch.full((B,), -7, dtype=torch.int32, device=DEV),
           "path": torch.full((B, max(tree.depth, 1)), -7, dtype=torch.int32, device=DEV),
           "final_token": torch.full((B,), -7, dtype=torch.int32, device=DEV),
           "decision": torch.full((B, M), 9, dtype=torch.uint8, device=DEV),
           "ratio": torch.zeros((B, M), device=DEV), "mass": torch.zeros((B, M), device=DEV),
           "n_agg": torch.zeros((B, M), dtype=torch.int32, device=DEV),
           "q_tok": torch.zeros((B, M), device=DEV), "p_tok": torch.zeros((B, M), device=DEV),
           "final_tok_all": torch.full((B, M), -7, dtype=torch.int32, device=DEV)}
    ws = torch.empty(lpp.lpp_relaxed_verify_workspace(tree, B, V, k), dtype=torch.uint8, device=DEV)
    lpp.lpp_relaxed_verify_opts(tree, dev(x["target_logits"]), dev(x["drafter_logits"]), cfg.ldv, off, V, B,
                                dev(x["tokens"]), dev(neigh), neigh.shape[1], k, dev(x["u_accept"]), dev(x["u_final"]),
                                out, ws, bound=lpp.LPP_BOUND_ADDITIVE if additive else lpp.LPP_BOUND_MULTIPLICATIVE,
                                bound_value=lam, rule=lpp.LPP_RULE_SKIP, siblings=lpp.LPP_SIBLINGS_DISTINCT,
                                uncond_logits=dev(y["target_logits"]), cfg_scale=3.0, top_k=2000)
    torch.cuda.synchronize()
    got = {n: t.cpu().numpy() for n, t in out.items()}
    filt = sampling_frontend(x["target_logits"], y["target_logits"], 3.0, 2000, off, V)
    rep = compare_verify(parent, dict(x, target_logits=filt), neigh, V, off, k, lam, got, additive=additive,
                         rule="skip", siblings="without_replacement")
    print(f"front end + skip + distinct, additive={additive}: {rep}", flush=True)
    assert rep["nodes"] > 0 and rep["near_tie_decisions"] <= 2


@pytest.mark.parametrize("idx", [1, 3])
def test_opts_builds_take_turns_on_one_handle(idx):
    # with every row's block resident the walk goes through the handle's words whatever the options: the builds in
    # turn on one handle, with other inputs each, give what each gives on a handle of its own; a walk that gives up
    # says so (the plain step) or is handed over to another row (calls with options, whose walks never end without a
    # result), and harms no later call of another build
    cfg = CONFIGS[idx]
    parent = static_tree(cfg.branching, cfg.N)
    E = make_codebook(cfg)
    skip, distinct, front = dict(rule=lpp.LPP_RULE_SKIP), dict(siblings=lpp.LPP_SIBLINGS_DISTINCT), dict(top_k=cfg.V // 8)
    builds = [None, skip, distinct, front, dict(**front, **distinct), dict(**front, **skip, **distinct)]
    xs = [make_verify_inputs(cfg, parent, rho=0.8, salt=s) for s in range(len(builds))]
    neigh = sparse_neighbour_table(E, cfg.k, np.concatenate([x["tokens"][:, 1:].ravel() for x in xs]), cfg.V)

    def call(tree, i):
        return run_verify(tree, xs[i], neigh, cfg.V, cfg.vocab_offset, cfg.ldv, cfg.k, cfg.lam, opts=builds[i])

    want = [call(lpp.Tree(parent), i) for i in range(len(builds))]
    tree = lpp.Tree(parent)
    for i in (0, 1, 2, 3, 4, 5, 3, 1, 0, 5, 2):
        got = call(tree, i)
        for n in got:
            assert np.array_equal(got[n], want[i][n], equal_nan=True), (i, n)
    for i in range(len(builds)):
        tree.set_walk_patience(-1)
        got = call(tree, i)
        if builds[i] is None:
            assert np.all(got["accept_len"] == -1) and np.all(got["final_token"] == -1) and np.all(got["path"] == -1)
            assert np.array_equal(got["decision"], want[i]["decision"])
        else:
            for n in got:
                assert np.array_equal(got[n], want[i][n], equal_nan=True), (i, n)
        tree.set_walk_patience(1 << 19)
        j = (i + 2) % len(builds)
        got = call(tree, j)
        for n in got:
            assert np.array_equal(got[n], want[j][n], equal_nan=True), (i, j, n)
    assert tree.walk_gave_up() == cfg.B


# (wide: a root with more than 64 children, whose words several waves write; alone: no row but the root)
@pytest.mark.parametrize("shape", ["B1", "B4", "wide", "alone"])
@pytest.mark.parametrize("opts", [dict(siblings=lpp.LPP_SIBLINGS_DISTINCT), dict(top_k=300),
                                  dict(rule=lpp.LPP_RULE_SKIP, siblings=lpp.LPP_SIBLINGS_DISTINCT, top_k=300)])
def test_opts_a_walk_that_gives_up_is_handed_over(shape, opts):
    # however early the walking block gives up (at once, after a few rounds, while the last rows finish), call after
    # call on one handle, with the full wait in between: every output as without
    cfg = CONFIGS[1].scaled(V=2000, ldv=2000, k=50) if shape in ("wide", "alone") else CONFIGS[3].scaled(B=int(shape[1]))
    parent = {"wide": np.array([-1] + [0] * 100 + list(range(1, 101)), dtype=np.int32), "alone": np.array([-1], dtype=np.int32)}.get(
        shape, static_tree(cfg.branching, cfg.N))
    cfg = cfg.scaled(N=len(parent) - 1)
    x = make_verify_inputs(cfg, parent, rho=0.8)
    neigh = sparse_neighbour_table(make_codebook(cfg), cfg.k, x["tokens"].ravel(), cfg.V)
    tree = lpp.Tree(parent)

    def call():
        return run_verify(tree, x, neigh, cfg.V, cfg.vocab_offset, cfg.ldv, cfg.k, cfg.lam, opts=opts)

    want = call()
    assert np.all(want["accept_len"] >= 0)
    for rounds in (-1, 0, 1, 2, 4, 8, 12, 16, 20, 24, 28, 32, -1, 1 << 19, -1, 3, 1 << 19):
        tree.set_walk_patience(rounds)
        got = call()
        for n in got:
            assert np.array_equal(got[n], want[n], equal_nan=True), (rounds, n)
    assert tree.walk_gave_up() == 0


@pytest.mark.parametrize("opts", [dict(siblings=lpp.LPP_SIBLINGS_DISTINCT), dict(rule=lpp.LPP_RULE_SKIP), dict(top_k=2000),
                                  dict(rule=lpp.LPP_RULE_SKIP, siblings=lpp.LPP_SIBLINGS_DISTINCT, top_k=2000)])
@pytest.mark.parametrize("V,off", [(16384, 0), (5003, 3), (20000, 0)])
def test_opts_an_item_does_not_depend_on_its_batch(V, off, opts):
    # 4 items of 61 rows are resident at once, 5 are not: another build, the same bits
    cfg = CONFIGS[3].scaled(B=5, V=V, vocab_offset=off, ldv=V + off, k=700)
    parent = static_tree(cfg.branching, cfg.N)
    x = make_verify_inputs(cfg, parent, rho=0.8)
    neigh = sparse_neighbour_table(make_codebook(cfg), cfg.k, x["tokens"][:, 1:], V)
    tree = lpp.Tree(parent)
    five, four = [run_verify(tree, {n: t[:B] for n, t in x.items()}, neigh, V, off, cfg.ldv, cfg.k, cfg.lam, opts=opts) for B in (5, 4)]
    for n in four:
        assert np.array_equal(four[n], five[n][:4], equal_nan=True), n
