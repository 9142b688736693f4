"""GPU: the expert FFN on every tile the launch rule can choose, in each of its four launches, at sizes that fall between
tiles: row counts around a tile edge, d_model and d_ff that are no multiple of a tile or a slab, experts without rows.
The tile that the rule chooses for a shape is asserted, so that a shape cannot come to test another kernel unnoticed."""
import numpy as np
import pytest
import torch

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu

F, H = I.F32, I.BF16
S32, S64, S128, S256, P64, P128 = (32, 1), (64, 1), (128, 1), (256, 1), (64, 2), (128, 2)      # tile side, wave groups
#        name          T     d     f   E  k  capacity dtype, tiles of xd W1, h W2, dz with dW2, dxd with dW1
SHAPES = [
    ("bf16_64_one_row",    3,   72,  136,  3, 1,    1, H, [S64, S64, S64, S64]),       # nearly every row masked
    ("bf16_64_edge",     390,   64,  200,  3, 2,  129, H, [S64, S64, S64, S64]),       # rows past two 64-row tiles
    ("bf16_64_long_k",   120,  520, 1032,  4, 1,   40, H, [S64, S64, S64, S64]),       # slabs beyond the ring, last one partial
    ("bf16_128_few",    6400,  136, 1032, 64, 1,  127, H, [S128, S64, S128, S128]),    # few rows per expert, many tiles
    ("bf16_128_rows",   1500,  776, 2056,  4, 2,  800, H, [S128, S128, S256, S256]),   # the large tile leaves CUs idle
    ("bf16_256_ragged", 2600,  520, 2056,  8, 2,  700, H, [S256, S128, S128, S128]),   # both extents ragged
    ("bf16_256_second", 7168,  520,  328,  8, 2, 1900, H, [S128, S256, S128, S256]),   # h W2 with a partial last slab
    ("f32_32_edge",      390,   72,  200,  3, 2,  129, F, [S32, S32, S32, S32]),
    ("f32_32_long_k",    130,  328,  520,  2, 1,   65, F, [S32, S32, S32, S32]),
    ("f32_64_edge",     3084,  232,  232, 12, 1,  257, F, [P64, P64, P64, P64]),       # a row past four tiles, 40 columns past three
    ("f32_64_long_k",   1540,  456,  456,  4, 1,  385, F, [P64, P64, P64, P64]),       # partial last slabs of longer reductions
    ("f32_64_even",     3000,  256,  256, 10, 1,  300, F, [P64, P64, P64, P64]),       # whole slabs
    ("f32_64_table_1",  2145,   24,  192, 65, 1,   33, F, [P64, S32, P128, P128]),     # more experts than lanes
    ("f32_64_table_2",  2145,  192,   24, 65, 1,   33, F, [S32, P64, P128, P128]),
    ("f32_64_table_3",  6790,   72,   72, 70, 1,   97, F, [S32, S32, P64, P64]),
    ("f32_64_table_4",  2145,  128,  128, 65, 1,   33, F, [S32, S32, P64, P64]),       # and whole slabs
    ("f32_128_groups",  1500,  136, 1032,  8, 2,  380, F, [P128, S32, P128, P64]),     # two wave groups per tile
    ("f32_128_single",  2200,   40, 2056,  8, 2,  560, F, [S128, S32, P128, S32]),
    ("f32_128_one",     8320,  264, 1032, 32, 2,  520, F, [S128, S128, S128, S128]),   # one group, partial last slabs
    ("f32_128_one_even", 8320, 272, 1040, 32, 2,  520, F, [S128, S128, S128, S128]),   # whole slabs
]


def test_the_shapes_cover_every_tile_of_every_launch():
    for dtype, tiles in ((H, {S64, S128, S256}), (F, {S32, P64, P128, S128})):
        for launch in range(4):
            seen = {s[8][launch] for s in SHAPES if s[7] == dtype}
            # fp32's two-group tile in h W2 and in dxd + dW1: with the accuracy of the fp32 products
            assert seen >= tiles - ({P128} if dtype == F and launch in (1, 3) else set()), (dtype, launch, seen)


@pytest.mark.parametrize("name,T,d,f,E,k,C,dtype,tiles", SHAPES, ids=[s[0] for s in SHAPES])
@pytest.mark.parametrize("act", [I.GELU, I.RELU], ids=["gelu", "relu"])
def test_ffn_tile(name, T, d, f, E, k, C, dtype, tiles, act):
    assert B.moe_expert_ffn_tiles(B.make_shape(T, d, f, E, k, C, dtype, act)) == tiles
    w = I.small(name, T, d, f, E, k, C, dtype, act, skew="hot0" if E > 2 else "none", skew_param=0.4)
    # ReLU's derivative jumps at 0.  The fp32 products are within 1e-6 of the exact ones (3e-7 measured), relative to their
    # standard deviation; with seed 5 no sum of the f32_64 shapes is nearer to 0 than 1.4e-6 of it (with seed 3 one is at 4e-8).
    data = I.make_inputs(w, seed=5 if name.startswith("f32_64") else 3)
    _, got = G.run_layer(w, data)
    G.check_full(w, data, got)


@pytest.mark.parametrize("dtype", [F, H], ids=["f32", "bf16"])
@pytest.mark.parametrize("E,C,d,f", [(5, 40, 72, 136), (100, 8, 200, 520), (40, 3, 136, 2056)])
def test_experts_without_rows_get_zero_weight_gradients(E, C, d, f, dtype):
    rng = np.random.default_rng(E)
    cnt = np.where(np.arange(E) % 3 == 1, rng.integers(1, C + 1, E), 0).astype(np.int32)
    tdt = torch.bfloat16 if dtype == H else torch.float32
    xd, h, dact, dyd = (torch.from_numpy(rng.standard_normal((E, C, n)).astype(np.float32)).cuda().to(tdt) for n in (d, f, f, d))
    W1, W2 = (torch.from_numpy(0.05 * rng.standard_normal((E, *n)).astype(np.float32)).cuda().to(tdt) for n in ((d, f), (f, d)))
    s = B.make_shape(E * C, d, f, E, 1, C, dtype, I.GELU)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    dxd, dW1, dW2 = torch.empty_like(xd), torch.full((E, d, f), float("nan"), device="cuda"), torch.full((E, f, d), float("nan"), device="cuda")
    print(f"[gpu] ffn backward with empty experts E={E} C={C} d={d} f={f} dtype={dtype}", flush=True)
    B.moe_expert_ffn_bwd(s, dyd, xd, h, dact, G.to_dev(cnt, None), W1, W2, dxd, dW1, dW2, ws)
    torch.cuda.synchronize()
    dW1, dW2 = G.host(dW1), G.host(dW2)
    for e in range(E):
        n = cnt[e]
        if n == 0:
            assert not dW1[e].any() and not dW2[e].any(), e
            continue
        X, D, Hh, A, V2 = (G.host(t[e]).astype(np.float64) for t in (xd, dyd, h, dact, W2))
        dz = (D[:n] @ V2.T) * A[:n]
        assert G.rel_l2(dW2[e], Hh[:n].T @ D[:n]) <= 1e-5           # fp32 sums of products of given values
        assert G.rel_l2(dW1[e], X[:n].T @ dz) <= G.TOL[dtype]       # dz is stored in the activation type
