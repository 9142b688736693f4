"""GPU: error of the fp32 GeLU and its derivative against 64 bits, on the forward FFN's epilogue.  W1 is the identity, so
the pre-activation is the input itself, exactly."""
import math

import numpy as np
import pytest
import torch
from scipy.special import erfc

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu

# rms error of h and of h' with erff and expf (0.5 (1 + erff(z / sqrt 2)), z phi(z)) on this GPU: the bounds
RANGES = [(0.0, 0.5, 7.4e-9, 2.57e-8), (-0.5, 0.0, 4.41e-9, 1.39e-8), (0.5, 1.0, 2.39e-8, 3.66e-8), (-1.0, -0.5, 1.16e-8, 1.56e-8),
          (1.0, 1.5, 4.41e-8, 4.37e-8), (-1.5, -1.0, 1.91e-8, 1.76e-8), (1.5, 2.0, 5.24e-8, 4.22e-8), (-2.0, -1.5, 1.87e-8, 1.44e-8),
          (2.0, 3.0, 8.88e-8, 4.14e-8), (-3.0, -2.0, 2.27e-8, 9.97e-9), (3.0, 5.0, 1.43e-7, 4.13e-8), (-5.0, -3.0, 3.47e-8, 8.62e-9),
          (5.0, 8.0, 7.73e-8, 2.41e-8), (-8.0, -5.0, 2.43e-8, 4.50e-9)]


def gelu32(z):
    C, d = z.shape
    s = B.make_shape(C, d, d, 1, 1, C, I.F32, I.GELU)
    eye = torch.eye(d, device="cuda")[None].contiguous()
    h, a, yd = (torch.empty(1, C, d, device="cuda") for _ in range(3))
    B.moe_expert_ffn_fwd(s, G.to_dev(z[None], I.F32), torch.tensor([C], dtype=torch.int32, device="cuda"), eye, eye, h, a, yd)
    torch.cuda.synchronize()
    return G.host(h)[0].astype(np.float64), G.host(a)[0].astype(np.float64)


@pytest.mark.parametrize("lo,hi,rms_h,rms_a", RANGES)
def test_gelu_error(lo, hi, rms_h, rms_a):
    z = np.random.default_rng(0).uniform(lo, hi, (16384, 64)).astype(np.float32)
    print(f"[gpu] fp32 gelu on [{lo}, {hi}]", flush=True)
    h, a = gelu32(z)
    z64 = z.astype(np.float64)
    cdf = 0.5 * erfc(-z64 / math.sqrt(2.0))
    eh, ea = h - z64 * cdf, a - (cdf + z64 * np.exp(-0.5 * z64 * z64) / math.sqrt(2.0 * math.pi))
    # 1 %: the bounds above are rounded and of another sample
    assert np.sqrt((eh ** 2).mean()) <= 1.01 * rms_h
    assert np.sqrt((ea ** 2).mean()) <= 1.01 * rms_a


def test_gelu_far_out():
    """Large and infinite pre-activations: h and h' are z and 1 on the right, 0 on the left; -inf gives 0 * inf = NaN."""
    z = np.array([13.0, 16.0, 40.0, 1e19, 3e38, -13.5, -16.0, -40.0, -1e19, -3e38], np.float32)
    h, a = gelu32(np.resize(z, (64, 8)))
    want = np.resize(np.maximum(z, 0).astype(np.float64), (64, 8))
    assert np.abs(h - want).max() <= 1e-36
    assert np.abs(a - (want > 0)).max() <= 1e-36
