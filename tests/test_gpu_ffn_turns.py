"""GPU: the backward's launches of two products where the second one's tiles are dealt unevenly: workgroups without a
tile in the first product's last round take several rounds of the second's first, then all take turns again.  On each
kernel and each way to find a tile; every output against the oracle, so that a tile left out or taken for another shows."""
import pytest

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu

# rounds: of dz with dW2 and of dxd with dW1, those that workgroups without a tile in the first product's last round take of
# the second's before all take turns; 0 where no such turns are taken (one round holds all), 1 = evenly dealt
# name            T      d     f    E  k  capacity dtype   tile side of dz with dW2, of dxd with dW1   rounds
SHAPES = [
    ("large",     30000, 256, 1024, 120, 1, 256, I.BF16, (256, 256), (2, 3)),
    ("128_regs",   6400, 136, 1032,  64, 1, 127, I.BF16, (128, 128), (2, 4)),
    ("128_table",  6400, 136, 1032,  70, 1, 127, I.BF16, (128, 128), (2, 4)),
    ("128_one_round", 16384, 256, 256, 2, 1, 8300, I.BF16, (128, 128), (0, 0)),     # more tiles than CUs, fewer than run at once
    ("64",          600, 512, 2048,  10, 1,  60, I.BF16, (128, 64), (3, 7)),
    ("64_table",   1300, 136,  264,  65, 1,  20, I.BF16, (64, 64), (2, 2)),
    ("f32_64",      320, 264,  264,  16, 1,  20, I.F32, (64, 64), (2, 2)),
    ("f32_64_32",  8000, 120,  232,   5, 1, 1600, I.F32, (64, 32), (1, 0)),
    ("f32_128_64", 1500, 136, 1032,   8, 2, 380, I.F32, (128, 64), (1, 3)),
    ("f32_128_groups", 320, 136, 1032, 16, 1, 20, I.F32, (128, 128), (2, 5)),
    ("f32_128_groups_table", 1300, 136, 136, 65, 1, 20, I.F32, (128, 128), (2, 2)),
    ("f32_128",     480, 136, 2056,  24, 1,  20, I.F32, (128, 128), (2, 8)),
    ("f32_128_table", 1400, 136, 520, 70, 1, 20, I.F32, (128, 128), (2, 3)),
    ("f32_32_table", 260,  64,   64, 65, 1,   4, I.F32, (32, 32), (2, 2)),
    ("64_hot",     1936, 384,  816,  16, 1, 968, I.BF16, (64, 64), (2, 2)),       # 2 and 3 by the rows to be expected
    ("f32_128_eighth", 330, 368, 1424, 14, 1, 48, I.F32, (128, 128), (3, 6)),     # 1.92 and 4.95 tiles
]


def rounds_first(s, launch, count):
    """What the walk makes of these row counts, as the dealing is described beside it."""
    side, _ = B.moe_expert_ffn_tiles(s)[launch]
    if B.moe_expert_ffn_direct(s)[launch]:
        return 0
    d, f, E = s.d_model, s.d_ff, s.E
    N, L = (f, d) if launch == 2 else (d, f)
    c = lambda x: -(-int(x) // side)
    first, second = sum(c(n) for n in count) * c(N), E * c(f) * c(d)
    per_xcd = B.moe_expert_ffn_workgroups(s)[launch] // 8
    by_table = E > 64 or side == 256
    if not by_table and -(-first // 8) - (-second // 8) <= per_xcd:
        return 0
    step = 8 * min(per_xcd, -(-(first + second) // 8))
    if first % step == 0:
        return 1
    tile = int(max(count)) + 300            # the expert with the most rows has the longest tiles: an eighth more counts
    return (L + 300 + tile + tile // 8 - 1) // tile


@pytest.mark.parametrize("name,T,d,f,E,k,C,dtype,sides,rounds", SHAPES, ids=[s[0] for s in SHAPES])
def test_second_product_of_a_launch(name, T, d, f, E, k, C, dtype, sides, rounds):
    s = B.make_shape(T, d, f, E, k, C, dtype, I.RELU)
    assert tuple(t[0] for t in B.moe_expert_ffn_tiles(s)[2:]) == sides
    w = I.small(name, T, d, f, E, k, C, dtype, I.RELU, skew="hot0", skew_param=0.2 if E < 50 else 0.02)
    data = I.make_inputs(w, seed=9)
    _, got = G.run_layer(w, data)
    assert tuple(rounds_first(s, i, got["expert_count"]) for i in (2, 3)) == rounds
    G.check_full(w, data, got)


def test_the_shapes_reach_uneven_turns_on_every_kernel():
    uneven = {(s[7], side, s[4] > 64) for s in SHAPES for side, r in zip(s[8], s[9]) if r > 1}
    assert uneven >= {(I.BF16, 256, True), (I.BF16, 128, False), (I.BF16, 128, True), (I.BF16, 64, False), (I.BF16, 64, True),
                      (I.F32, 128, False), (I.F32, 128, True), (I.F32, 64, False), (I.F32, 32, True)}
