"""GPU: the smallest fp32 products, as 32 x 32 tiles whose reduction four waves share, in each of the three ways in which a
workgroup finds its tile: addressed without the experts' row counts (buffers that are mostly full, a CU for each tile), from
counts held in registers (half-empty buffers, up to 64 experts) and from the table in LDS (more experts); and as 64 x 64
ones by the first two (by the table: in the test of every tile)."""
import numpy as np
import pytest
import torch

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G
import test_gpu_ffn_range as R

pytestmark = pytest.mark.gpu

# name                T     d    f   E  k  capacity  32 x 32 tiles in xd W1, h W2, dz with dW2, dxd with dW1
SHAPES = [
    ("one_row",        1,    8,   8,  1, 1,   1, [True] * 4),                        # one chunk, one row and 8 columns in use
    ("full",          96,   32,  64,  3, 1,  32, [True] * 4),                        # whole tiles and chunks
    ("edges",        131,   40,  72,  4, 1,  33, [True] * 4),                        # a row, 8 columns and 8 entries of the reduction past them
    ("long_k",        60,  264, 296,  2, 1,  30, [True] * 4),                        # a wave takes several chunks, the last ones apart
    ("half_empty",   300,   72, 136,  5, 2, 240, [True] * 4),                        # counts in registers
    ("64_experts",   640,   24,  40, 64, 1,  40, [True] * 4),
    ("65_experts",   650,   24,  40, 65, 1,  40, [True] * 4),                        # counts in the table
    ("mixed",        520,  232, 832,  5, 2, 416, [True, True, False, True]),
    ("64_x_64",     3000,  232, 232, 10, 1, 300, [False] * 4),
    ("64_x_64_half", 3000, 232, 232, 10, 1, 600, [False] * 4),
]


@pytest.mark.parametrize("name,T,d,f,E,k,C,parts", SHAPES, ids=[s[0] for s in SHAPES])
def test_small_fp32_products(name, T, d, f, E, k, C, parts):
    s = B.make_shape(T, d, f, E, k, C, I.F32, I.GELU)
    assert [t[0] for t in B.moe_expert_ffn_tiles(s)] == [32 if p else 64 for p in parts] and B.moe_expert_ffn_parts(s) == parts
    w = I.small(name, T, d, f, E, k, C, I.F32, I.GELU, skew="hot0" if E > 2 else "none", skew_param=0.4)
    data = I.make_inputs(w, seed=5)
    _, got = G.run_layer(w, data)
    G.check_full(w, data, got)


@pytest.mark.parametrize("what", ["inf_row", "inf_weight", "nan", "large", "tiny"])
def test_operands_outside_the_exact_range_on_64_x_64_tiles(what):
    E, C, d, f = 10, 300, 232, 232
    assert not any(B.moe_expert_ffn_parts(B.make_shape(E * C, d, f, E, 1, C, I.F32, I.RELU)))
    R.test_fp32_operands_outside_the_exact_range(E, C, d, f, what, I.RELU)


def test_what_lies_behind_the_rows_in_use_does_not_matter():
    """Loads of the tiles that are addressed without the row counts may touch unused rows; whatever is there (NaN and
    infinities here) must neither change a result nor be written over."""
    E, C, d, f = 4, 40, 72, 136
    cnt = np.array([40, 33, 1, 0], np.int32)
    s = B.make_shape(E * C, d, f, E, 1, C, I.F32, I.GELU)
    assert all(B.moe_expert_ffn_parts(s))
    rng = np.random.default_rng(7)
    host = {n: rng.standard_normal((E, C, m)).astype(np.float32) for n, m in (("xd", d), ("dyd", d))}
    W1, W2 = (0.1 * rng.standard_normal((E, *m)).astype(np.float32) for m in ((d, f), (f, d)))
    outs = []
    for fill in (0.0, float("nan"), float("inf")):
        for n in host:
            for e in range(E):
                host[n][e, cnt[e]:] = fill
        new = lambda m: torch.full((E, C, m), fill, device="cuda")
        h, a, yd, dxd = new(f), new(f), new(d), new(d)
        dW1, dW2 = torch.empty(E, d, f, device="cuda"), torch.empty(E, f, d, device="cuda")
        ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
        ws.view(torch.float32).fill_(fill)
        c = G.to_dev(cnt, None)
        print(f"[gpu] unused rows hold {fill}", flush=True)
        B.moe_expert_ffn_fwd(s, G.to_dev(host["xd"], I.F32), c, G.to_dev(W1, I.F32), G.to_dev(W2, I.F32), h, a, yd)
        B.moe_expert_ffn_bwd(s, G.to_dev(host["dyd"], I.F32), G.to_dev(host["xd"], I.F32), h, a, c, G.to_dev(W1, I.F32), G.to_dev(W2, I.F32), dxd, dW1, dW2, ws)
        torch.cuda.synchronize()
        got = [G.host(t) for t in (h, a, yd, dxd, dW1, dW2)]
        for t in got[:4]:
            for e in range(E):
                assert np.array_equal(t[e, cnt[e]:], np.full_like(t[e, cnt[e]:], fill), equal_nan=True)
        outs.append([np.concatenate([t[e, :cnt[e]].ravel() for e in range(E)]) for t in got[:4]] + got[4:])
    for o in outs[1:]:
        for x, y in zip(outs[0], o):
            assert np.isfinite(x).all() and np.array_equal(x, y)


def test_more_tiles_than_workgroups():
    """A workgroup of the 32 x 32 kernel takes several tiles: row counts far above what the shape lets the rule expect (a
    routing call never writes such; every index stays inside the buffers).  Its sums in LDS are used again by each tile."""
    T, E, C, d, f = 64, 4, 1024, 256, 1032
    s = B.make_shape(T, d, f, E, 1, C, I.F32, I.RELU)
    assert B.moe_expert_ffn_tiles(s) == [(32, 1)] * 4 and not any(B.moe_expert_ffn_direct(s))
    cnt = np.array([1024, 1000, 1, 993], np.int32)
    tiles = sum(-(-int(n) // 32) for n in cnt)
    assert tiles * -(-f // 32) > 2048       # eight workgroups on each of 256 compute units
    rng = np.random.default_rng(3)
    normal = lambda *sh: rng.standard_normal(sh, dtype=np.float32)
    xd, dyd, hs, da, W1, W2 = normal(E, C, d), normal(E, C, d), normal(E, C, f), normal(E, C, f), normal(E, d, f), normal(E, f, d)
    dev = [G.to_dev(v, I.F32) for v in (xd, dyd, hs, da, W1, W2)]
    c = G.to_dev(cnt, None)
    h, a, yd, dxd, dW1, dW2 = (torch.zeros(E, m, n, device="cuda") for m, n in ((C, f), (C, f), (C, d), (C, d), (d, f), (f, d)))
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    print("[gpu] 32 x 32 tiles in several rounds", flush=True)
    B.moe_expert_ffn_fwd(s, dev[0], c, dev[4], dev[5], h, a, yd)
    B.moe_expert_ffn_bwd(s, dev[1], dev[0], dev[2], dev[3], c, dev[4], dev[5], dxd, dW1, dW2, ws)
    dz = ws[:E * C * f * 4].view(torch.float32).view(E, C, f)       # the workspace holds dz
    torch.cuda.synchronize()
    got = {n: G.host(t) for n, t in (("h", h), ("yd", yd), ("dz", dz), ("dxd", dxd), ("dW1", dW1), ("dW2", dW2))}
    for e in range(E):
        n = cnt[e]
        x, dy, hh, dd, w1, w2 = (v[e].astype(np.float64) for v in (xd, dyd, hs, da, W1, W2))
        hg, dzg = got["h"][e][:n].astype(np.float64), got["dz"][e][:n].astype(np.float64)
        want = {"h": np.maximum(x[:n] @ w1, 0.0), "yd": hg @ w2, "dz": (dy[:n] @ w2.T) * dd[:n], "dxd": dzg @ w1.T,
                "dW1": x[:n].T @ dzg, "dW2": hh[:n].T @ dy[:n]}
        for name, w in want.items():
            g = got[name][e] if "W" in name else got[name][e][:n]
            # the bound of the fp32 products: any of their six parts that is missing is twice as far off
            assert G.rel_l2(g, w) <= 1e-6, (name, e, G.rel_l2(g, w))
            assert float(np.abs(g - w).max()) <= 1e-4 * float(np.abs(w).max()), (name, e)
