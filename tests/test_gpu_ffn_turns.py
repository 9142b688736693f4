"""GPU: the backward's launches of two products where the second one's tiles are dealt unevenly: workgroups without a
tile in the first product's last round take several rounds of the second's first, then all take turns again.  On each
kernel and each way to find a tile; every output against the oracle, so that a tile left out or taken for another shows."""
import pytest

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu

# name            T      d     f    E  k  capacity dtype   tile side of dz with dW2, of dxd with dW1
SHAPES = [
    ("large",     30000, 256, 1024, 120, 1, 256, I.BF16, (256, 256)),
    ("128_regs",   6400, 136, 1032,  64, 1, 127, I.BF16, (128, 128)),
    ("128_one_round", 16384, 256, 256, 2, 1, 8300, I.BF16, (128, 128)),     # more tiles than CUs, fewer than run at once
    ("128_table",  6400, 136, 1032,  70, 1, 127, I.BF16, (128, 128)),
    ("64",          600, 512, 2048,  10, 1,  60, I.BF16, (128, 64)),
    ("f32_64_32",  8000, 120,  232,   5, 1, 1600, I.F32, (64, 32)),
    ("f32_128",    1500, 136, 1032,   8, 2, 380, I.F32, (128, 64)),
]


@pytest.mark.parametrize("name,T,d,f,E,k,C,dtype,sides", SHAPES, ids=[s[0] for s in SHAPES])
def test_second_product_of_a_launch(name, T, d, f, E, k, C, dtype, sides):
    s = B.make_shape(T, d, f, E, k, C, dtype, I.RELU)
    assert tuple(t[0] for t in B.moe_expert_ffn_tiles(s)[2:]) == sides
    w = I.small(name, T, d, f, E, k, C, dtype, I.RELU, skew="hot0", skew_param=0.2 if E < 50 else 0.02)
    data = I.make_inputs(w, seed=9)
    _, got = G.run_layer(w, data)
    G.check_full(w, data, got)
