"""The fp32 expert FFN is accurate to fp32: its products are six partial products of bf16 parts, and a result from which
any one of them is missing is at least 2.4e-6 away from the exact one.  The GPU's results are held to 1e-6, each product
by itself: operands are given, no rounded intermediate lies between."""
import numpy as np
import pytest
import torch

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

#         E    C    d     f  tile (side, wave groups) of xd W1, h W2, dz with dW2, dxd with dW1
SHAPES = [(2, 70, 72, 136, [(32, 1)] * 4),
          (12, 257, 232, 232, [(64, 2)] * 4),
          (10, 300, 256, 256, [(64, 2)] * 4),           # reductions without a partial slab
          (8, 380, 136, 1032, [(128, 2), (32, 1), (128, 2), (64, 2)]),
          (8, 380, 904, 1032, [(128, 2)] * 4),
          (32, 520, 264, 1032, [(128, 1)] * 4),
          (32, 520, 272, 1040, [(128, 1)] * 4)]       # reductions without a partial slab
BOUND = 1e-6


def bf16(x):
    return I.round_to_bf16(x.astype(np.float32))


def parts(x):
    hi = bf16(x)
    mid = bf16(x - hi)
    return [v.astype(np.float64) for v in (hi, mid, bf16(x - hi - mid))]


def test_the_bound_tells_a_missing_partial_product():
    """On the CPU: the six products together are far below the bound, any five of them more than twice above it."""
    rng = np.random.default_rng(0)
    a, w = rng.standard_normal((256, 512)).astype(np.float32), rng.standard_normal((512, 256)).astype(np.float32)
    exact = a.astype(np.float64) @ w.astype(np.float64)
    pa, pw = parts(a), parts(w)
    six = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]
    assert G.rel_l2(sum(pa[i] @ pw[j] for i, j in six), exact) <= 0.01 * BOUND
    for gone in six:
        assert G.rel_l2(sum(pa[i] @ pw[j] for i, j in six if (i, j) != gone), exact) >= 2.0 * BOUND, gone


@pytest.mark.gpu
@pytest.mark.parametrize("E,C,d,f,tiles", SHAPES, ids=lambda v: str(v) if isinstance(v, int) else "")
def test_fp32_products(E, C, d, f, tiles):
    s = B.make_shape(E * C, d, f, E, 1, C, I.F32, I.RELU)
    assert B.moe_expert_ffn_tiles(s) == tiles
    rng = np.random.default_rng(E + d)
    normal = lambda *sh: rng.standard_normal(sh, dtype=np.float32)
    xd, dyd, hs, da, W1, W2 = normal(E, C, d), normal(E, C, d), normal(E, C, f), normal(E, C, f), normal(E, d, f), normal(E, f, d)
    cnt = np.full(E, C, np.int32)
    cnt[0], cnt[-1] = C - 1, C - 35
    dev = [G.to_dev(v, I.F32) for v in (xd, dyd, hs, da, W1, W2)]
    c = G.to_dev(cnt, None)
    h, a, yd, dxd, dW1, dW2 = (torch.zeros(E, m, n, device="cuda") for m, n in ((C, f), (C, f), (C, d), (C, d), (d, f), (f, d)))
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    print(f"[gpu] fp32 products E={E} C={C} d={d} f={f}", flush=True)
    B.moe_expert_ffn_fwd(s, dev[0], c, dev[4], dev[5], h, a, yd)
    B.moe_expert_ffn_bwd(s, dev[1], dev[0], dev[2], dev[3], c, dev[4], dev[5], dxd, dW1, dW2, ws)
    dz = ws[:E * C * f * 4].view(torch.float32).view(E, C, f)       # the workspace holds dz
    torch.cuda.synchronize()
    got = {n: G.host(t) for n, t in (("h", h), ("yd", yd), ("dz", dz), ("dxd", dxd), ("dW1", dW1), ("dW2", dW2))}
    for e in sorted({0, E // 2, E - 1}):
        n = cnt[e]
        x, dy, hh, dd, w1, w2 = (v[e].astype(np.float64) for v in (xd, dyd, hs, da, W1, W2))
        hg, dzg = got["h"][e][:n].astype(np.float64), got["dz"][e][:n].astype(np.float64)
        want = {"h": np.maximum(x[:n] @ w1, 0.0), "yd": hg @ w2, "dz": (dy[:n] @ w2.T) * dd[:n], "dxd": dzg @ w1.T,
                "dW1": x[:n].T @ dzg, "dW2": hh[:n].T @ dy[:n]}
        for name, w in want.items():
            g = got[name][e][:n] if name[0] != "d" or name in ("dz", "dxd") else got[name][e]
            assert G.rel_l2(g, w) <= BOUND, (name, e, G.rel_l2(g, w))
