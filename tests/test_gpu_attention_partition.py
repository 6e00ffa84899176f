"""How the keys of a bf16 row fall to waves (lpp_tree_attention and its forms; Sec. 2.1, App. A.2): the kernel's arithmetic
replayed on the host for a stated number of waves and key ranges.  Each wave rounds its weights to bf16 against a reference of its own, so
another partition gives a result as far from this one as either is from float64: 7e-4 to 3e-3."""
import numpy as np
import pytest
import torch

import paper_2502_06352_amd as lpp
from workloads import static_tree
from gpu_common import DEV, dev

pytestmark = pytest.mark.gpu
MASKED, LIMIT = np.float32(-1e30), np.float32(8.0)


def _bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).float().numpy()


def _replay(q, kc, vc, kt, vt, vis, waves, ranges):
    """One head: q [M, Dh], kc and vc the item's cached rows.  Sums in float64, what the kernel rounds in float32 or bf16."""
    M, Dh = q.shape
    n = kc.shape[0]
    scale_log2 = np.float32(np.float32(1.0) / np.sqrt(np.float32(Dh))) * np.float32(1.44269504088896340736)
    # groups of 32 keys: those wholly in the cache, then its ragged end and the tree's
    groups = [(slice(g, min(g + 32, n)), True) for g in range(0, n, 32)] + [(slice(g, min(g + 32, M)), False) for g in range(0, M, 32)]
    full, G = n // 32, len(groups)
    sums = []
    for r in range(ranges):
        g0, g1 = r * G // ranges, (r + 1) * G // ranges
        for w in range(waves):
            mine = list(range(g0 + w, min(g1, full), waves))
            others = list(range(max(g0, full) + w, g1, waves))
            ref = np.full(M, MASKED, dtype=np.float32)
            o, l = np.zeros((M, Dh)), np.zeros(M)
            for g in others[:1] + mine + others[1:]:
                part, cached = groups[g]
                K, V = (kc[part], vc[part]) if cached else (kt[part], vt[part])
                s = (q.astype(np.float64) @ K.T.astype(np.float64)).astype(np.float32)
                seen = np.ones(s.shape, dtype=bool) if cached else vis[:, part]
                top = np.where(seen, s, MASKED).max(axis=1)
                top = np.where(top > 0.5 * MASKED, top * scale_log2, MASKED).astype(np.float32)
                new = np.where(top > ref + LIMIT, top, ref)
                with np.errstate(over="ignore"):
                    keep = np.exp2((ref - new).astype(np.float64))
                    p = np.exp2((s.astype(np.float64) * scale_log2 - new[:, None]).astype(np.float32).astype(np.float64))
                p = _bf16(np.where(seen, p, 0.0)).astype(np.float64)
                o, l, ref = o * keep[:, None] + p @ V, l * keep + p.sum(axis=1), new
            sums.append((ref.astype(np.float64), l, o))
    top = np.max([s[0] for s in sums], axis=0)
    f = [np.exp2(s[0] - top) for s in sums]
    return sum(x[:, None] * s[2] for x, s in zip(f, sums)) / sum(x * s[1] for x, s in zip(f, sums))[:, None]


@pytest.mark.parametrize("N,S,B,H,Hkv,Dh,L,ragged,waves,ranges", [
    (108, 270, 7, 20, 20, 64, 1, False, 8, 1),     # 280 blocks of four tiles
    (100, 1504, 5, 8, 8, 64, 1, False, 8, 3),      # few blocks: three ranges
    (120, 1914, 1, 20, 20, 64, 2, False, 8, 3),
    (12, 185, 4, 32, 32, 64, 10, False, 8, 1),     # one tile, blocks in many rounds
    (13, 160, 12, 12, 12, 64, 5, False, 8, 1),     # five full groups
    (13, 159, 12, 12, 12, 64, 5, True, 8, 1),      # four: blocks of 4 waves do
    (95, 128, 3, 16, 16, 64, 1, True, 8, 1),       # ... with four general groups at most
    (96, 128, 3, 16, 16, 64, 1, True, 8, 1),       # five
    (60, 200, 1, 16, 16, 64, 1, False, 8, 1),
    (26, 1024, 1, 16, 16, 64, 1, True, 8, 2),      # two ranges, two blocks of 4 waves for each
    (99, 1313, 1, 4, 1, 64, 1, False, 8, 2),
    (20, 2481, 1, 16, 16, 64, 1, False, 8, 4),
    (10, 4075, 1, 20, 20, 64, 1, False, 8, 8),     # eight, not shared
    (60, 2400, 1, 32, 8, 128, 1, False, 8, 4),
    (28, 282, 3, 32, 32, 128, 1, False, 8, 1),
    (60, 1024, 4, 24, 24, 64, 1, True, 8, 1),
    (30, 1100, 12, 24, 24, 64, 1, False, 4, 1),    # more blocks than compute units
    (60, 1024, 4, 24, 24, 64, 4, True, 4, 1),      # ... and all rows of a head in one
    (51, 246, 8, 20, 20, 64, 1, False, 4, 1),
    (45, 240, 8, 20, 20, 64, 1, False, 4, 1),
    (128, 1100, 12, 24, 8, 64, 1, False, 4, 1),
])
def test_keys_fall_to_waves_as_stated(N, S, B, H, Hkv, Dh, L, ragged, waves, ranges):
    parent = static_tree((8, 4, 2, 2, 1, 1, 1, 1), N)
    M = len(parent)
    vis = np.zeros((M, M), dtype=bool)
    for i in range(M):
        j = i
        while j >= 0:
            vis[i, j] = True
            j = parent[j]
    tree = lpp.Tree(parent)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(N + S)

    def normal(heads, rows):
        return torch.randn(B, heads, rows, Dh, generator=gen, device=DEV).to(torch.bfloat16)

    layers = [dict(q=normal(H, M), k_cache=normal(Hkv, S), v_cache=normal(Hkv, S), k_tree=normal(Hkv, M), v_tree=normal(Hkv, M),
                   out=torch.full((B, H, M, Dh), float("nan"), device=DEV)) for _ in range(L)]
    seq = [S - b * S // (2 * B) if ragged else S for b in range(B)]
    ws = torch.empty(lpp.lpp_tree_attention_layers_workspace(tree, L, B, H, S, Dh), dtype=torch.uint8, device=DEV)
    lpp.lpp_tree_attention_layers(tree, lpp.LPP_BF16, lpp.LPP_F32, layers, dev(np.asarray(seq, dtype=np.int32)) if ragged else None,
                                  B, H, Hkv, S, Dh, 0.0, ws)
    y = layers[-1]
    for b, h in {(0, 0), (B // 2, H // 2), (B - 1, H - 1)}:
        kv = h // (H // Hkv)
        x = [t.float().cpu().numpy() for t in (y["q"][b, h], y["k_cache"][b, kv, :seq[b]], y["v_cache"][b, kv, :seq[b]], y["k_tree"][b, kv],
                                               y["v_tree"][b, kv])]
        want = _replay(*x, vis, waves, ranges)
        got = y["out"][b, h].double().cpu().numpy()
        # A weight that float32 puts on the other side of a rounding to bf16 (one in about 10^4: exponents up to 10, off by a few
        # 2^-24 of it, against steps of 2^-9) differs by 2^-8: 1e-4 of a weight in the root of the squares, and many make a row's sum.
        assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want), (b, h)
