"""GPU: the expert FFN on every tile the launch rule can choose, at sizes that fall between tiles: row counts around
a tile edge, d_model and d_ff that are no multiple of a tile or a slab, experts without rows."""
import pytest

from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu

F, H = I.F32, I.BF16
#        name          T     d     f   E  k  capacity dtype
SHAPES = [
    ("bf16_64_one_row",    3,   72,  136,  3, 1,    1, H),     # 64 x 64, nearly every row masked
    ("bf16_64_edge",     390,   64,  200,  3, 2,  129, H),     # rows past two 64-row tiles
    ("bf16_64_long_k",   120,  520, 1032,  4, 1,   40, H),     # slabs beyond the ring, last one partial
    ("bf16_128_few",    6400,  136, 1032, 64, 1,  127, H),     # 128 x 128: few rows per expert, many tiles
    ("bf16_128_rows",   1500,  776, 2056,  4, 2,  800, H),     # 128 x 128 because the large tile leaves CUs idle
    ("bf16_256_ragged", 2600,  520, 2056,  8, 2,  700, H),     # the large tile, both extents ragged
    ("f32_64_edge",      390,   72,  200,  3, 2,  129, F),
    ("f32_64_long_k",    130,  328,  520,  2, 1,   65, F),
    ("f32_128_groups",  1500,  136, 1032,  8, 2,  380, F),     # 128 x 128, two wave groups per tile
    ("f32_128_single",  2200,   40, 2056,  8, 2,  560, F),     # 128 x 128, one group
]


@pytest.mark.parametrize("name,T,d,f,E,k,C,dtype", SHAPES, ids=[s[0] for s in SHAPES])
@pytest.mark.parametrize("act", [I.GELU, I.RELU], ids=["gelu", "relu"])
def test_ffn_tile(name, T, d, f, E, k, C, dtype, act):
    w = I.small(name, T, d, f, E, k, C, dtype, act, skew="hot0" if E > 2 else "none", skew_param=0.4)
    data = I.make_inputs(w, seed=3)
    _, got = G.run_layer(w, data)
    G.check_full(w, data, got)
