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
