"""GPU: the fp32 expert FFN on operands outside of the range in which its bf16 parts are exact - infinite and NaN values,
finite ones that round to infinity in bf16, and ones whose parts fall under bf16's subnormals - against the same
products in 64 bits, on each of the fp32 kernels."""
import math

import numpy as np
import pytest
import torch
from scipy.special import erfc

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu

#         E    C    d     f: tiles of 32 x 32; of 64 x 64; of 128 x 128 with two wave groups (in xd W1 and dz with dW2), with one
SHAPES = [(2, 70, 72, 136), (12, 257, 232, 232), (8, 380, 136, 1032), (16, 560, 520, 2056)]
TILES = [[(32, 1)] * 4, [(64, 2)] * 4, [(128, 2), (32, 1), (128, 2), (64, 2)], [(128, 1)] * 4]


def act64(z, act):
    with np.errstate(all="ignore"):
        if act == I.RELU:
            return np.fmax(z, 0.0), (z > 0).astype(np.float64)
        cdf = 0.5 * erfc(-z / math.sqrt(2.0))
        zpdf = z * np.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)
        return z * cdf, cdf + zpdf


def same(name, got, want, rel):
    """Infinities and NaN in the same places; the other values of the tensor within rel of each other (2-norm)."""
    with np.errstate(all="ignore"):
        want = want.astype(np.float32).astype(np.float64)
    got = got.astype(np.float64)
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)), (name, "NaN", int(np.isnan(got).sum()), int(np.isnan(want).sum()))
    assert np.array_equal(got[~fin], want[~fin], equal_nan=True), (name, "infinities")
    if fin.any():
        scale = max(float(np.abs(want[fin]).max()), 1e-300)      # norms of values near the type's ends
        assert G.rel_l2(got[fin] / scale, want[fin] / scale) <= rel, (name, G.rel_l2(got[fin] / scale, want[fin] / scale))


@pytest.mark.parametrize("act", [I.RELU, I.GELU], ids=["relu", "gelu"])
@pytest.mark.parametrize("what", ["inf_row", "inf_weight", "nan", "large", "tiny"])
@pytest.mark.parametrize("E,C,d,f", SHAPES, ids=["32", "64", "128x2", "128x1"])
def test_fp32_operands_outside_the_exact_range(E, C, d, f, what, act):
    rng = np.random.default_rng(E)
    std = 1.0 if what == "tiny" else 0.02
    xd, dyd = rng.standard_normal((E, C, d)).astype(np.float32), 0.1 * rng.standard_normal((E, C, d)).astype(np.float32)
    W1, W2 = std * rng.standard_normal((E, d, f)).astype(np.float32), std * rng.standard_normal((E, f, d)).astype(np.float32)
    cnt = np.full(E, C, np.int32)
    cnt[0], cnt[-1] = C - 1, C - 35
    if what == "inf_row":
        xd[0, 3, 5], dyd[E - 1, 7, 1] = np.inf, -np.inf
    elif what == "inf_weight":
        W1[0, 9, 2], W2[E - 1, 4, 6] = np.inf, -np.inf
    elif what == "nan":
        xd[0, 3, 5], W2[E - 1, 4, 6] = np.nan, np.nan
    elif what == "large":           # rounds to infinity in bf16; every result stays finite
        xd[0, 3, 5], xd[E - 1, 7, 1] = 3.395e38, -3.4e38
    else:
        xd *= np.float32(2.0 ** -122)
    s = B.make_shape(E * C, d, f, E, 1, C, I.F32, act)
    if (E, C, d, f) in SHAPES:
        assert B.moe_expert_ffn_tiles(s) == TILES[SHAPES.index((E, C, d, f))]
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    new = lambda *sh: torch.zeros(*sh, device="cuda")
    dx, dw1, dw2, ddy = (G.to_dev(a, I.F32) for a in (xd, W1, W2, dyd))
    c = G.to_dev(cnt, None)
    h, a, yd, dxd, dW1, dW2 = new(E, C, f), new(E, C, f), new(E, C, d), new(E, C, d), new(E, d, f), new(E, f, d)
    print(f"[gpu] fp32 FFN {what} E={E} C={C} d={d} f={f} act={act}", flush=True)
    B.moe_expert_ffn_fwd(s, dx, c, dw1, dw2, h, a, yd)
    h2 = new(E, C, f)
    B.moe_expert_ffn_fwd(s, dx, c, dw1, dw2, h2, None, new(E, C, d))
    B.moe_expert_ffn_bwd(s, ddy, dx, h, a, c, dw1, dw2, dxd, dW1, dW2, ws)
    torch.cuda.synchronize()
    got = {n: G.host(t) for n, t in (("h", h), ("h_eval", h2), ("dact", a), ("yd", yd), ("dxd", dxd), ("dW1", dW1), ("dW2", dW2))}
    # fp32 sums of up to 2056 products that cancel: the fp32 pipe is 1e-6 away, the split 3e-7
    rel = 5e-6
    for e in sorted({0, E // 2, E - 1}):
        n = cnt[e]
        X, D, A1, A2 = (v.astype(np.float64) for v in (xd[e, :n], dyd[e, :n], W1[e], W2[e]))
        with np.errstate(all="ignore"):
            z = X @ A1
            H, A = act64(z, act)
            if act == I.RELU:       # its derivative jumps at 0: within the products' rounding of it, take the kernel's side
                near = np.abs(z) <= 2e-6 * np.nanmedian(np.abs(z))
                A = np.where(near, got["dact"][e][:n], A)
            # what the kernels store in between is fp32
            H, A = H.astype(np.float32).astype(np.float64), A.astype(np.float32).astype(np.float64)
            dz = ((D @ A2.T) * A).astype(np.float32).astype(np.float64)
            want = {"h": H, "h_eval": H, "dact": A, "yd": H @ A2, "dxd": dz @ A1.T, "dW1": X.T @ dz, "dW2": H.T @ D}
        for name, w in want.items():
            same(f"{name}[{e}]", got[name][e][:n] if name not in ("dW1", "dW2") else got[name][e], w, rel)
