"""Which kernel the dispatch rules choose, at shapes where both sides have been measured (host-only queries).  The times in
the comments are microseconds on an MI355X."""
import pytest

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I


#        T     E   k  capacity keys  launches
ROUTE = [
    (61, 32, 1, 128, True, 1),          # one workgroup 9.1, three launches 15.5
    (61, 32, 1, 512, True, 1),          # 14.5, 15.4
    (61, 32, 1, 1024, True, 3),         # 21.8, 15.5
    (160, 32, 2, 10, True, 1),          # 13.7, 16.5
    (384, 32, 2, 24, True, 1),          # 16.4, 17.0
    (384, 32, 1, 12, False, 1),         # 12.1, 13.6
    (512, 32, 1, 16, True, 3),          # 18.0, 15.2
    (512, 32, 1, 16, False, 3),         # 15.0, 12.1
    (1024, 32, 2, 64, True, 3),         # 26.6, 16.6
    (512, 16, 1, 512, True, 1),         # 13.0, 14.7
    (512, 16, 1, 2048, True, 3),        # 18.1, 14.7
    (768, 16, 1, 48, True, 1),          # 13.1, 14.6
    (900, 16, 2, 112, True, 3),         # 16.6, 15.1
    (900, 16, 1, 56, False, 1),         # 9.8, 12.3
    (1024, 8, 1, 2048, True, 1),        # 13.3, 14.0
    (1024, 8, 1, 4096, True, 3),        # 15.9, 14.2
    (1024, 4, 1, 8192, True, 1),        # 14.2, 15.7
    (512, 8, 1, 4096, True, 3),         # 16.0, 14.3
    (90, 64, 2, 2, True, 1),            # 15.6, 20.0
    (256, 64, 1, 4, True, 3),           # 30.2, 19.3
    (64, 128, 1, 1, True, 1),           # 18.0, 19.9
    (64, 128, 1, 128, True, 3),         # 25.6, 20.1
    (128, 128, 2, 2, True, 3),          # 34.9, 23.0
    (24, 256, 1, 1, True, 1),           # 15.9, 21.5
    (64, 256, 1, 1, True, 3),           # 34.5, 22.1
    (1025, 4, 1, 256, True, 3),         # beyond one workgroup
]


@pytest.mark.parametrize("T,E,k,C,keys,launches", ROUTE)
def test_route(T, E, k, C, keys, launches):
    s = B.make_shape(T, 64, 64, E, k, C, I.BF16, I.GELU)
    assert B.moe_route_launches(s, 1, keys) == launches
    assert B.moe_route_launches(s, 2, keys) == 3            # groups are ranked on their own
    assert B.moe_route_launches(B.make_shape(T, 60, 64, E, k, C, I.BF16, I.GELU), 1, keys) == -2


@pytest.mark.parametrize("T,d,tiles", [
    (61, 1024, 1),          # one token tile per workgroup 5.1, two 6.8
    (61, 512, 2),           # 4.8, 4.7
    (61, 64, 2),            # 4.0, 3.5
    (4096, 640, 1),         # 5.5, 6.7
    (8192, 2048, 1),        # 10.5, 13.5
    (8256, 2048, 2),        # 16.3, 13.6
    (12224, 768, 2),        # 8.4, 7.1
    (12224, 256, 2),        # 8.0, 4.9
    (16384, 1024, 2)])      # 15.7, 14.2
def test_gate_projection(T, d, tiles):
    for E in (2, 8, 32):
        assert B.moe_gate_logits_token_tiles(B.make_shape(T, d, 64, E, 1, 8, I.BF16, I.GELU)) == tiles
    assert B.moe_gate_logits_token_tiles(B.make_shape(T, d, 64, 8, 1, 8, I.F32, I.GELU)) == 1


@pytest.mark.parametrize("T,d,E,with_dx,launches", [
    (1, 8, 1, True, 1),
    (512, 256, 32, False, 1),       # one launch 9.1, two 12.0
    (512, 8192, 32, True, 1),       # 53.6, three 57.1
    (512, 16384, 32, True, 3),      # 102.5, 100.1
    (512, 16384, 4, True, 1),       # 75.1, 81.5
    (1024, 256, 16, False, 1),      # 8.6, 13.1
    (1024, 8192, 16, True, 1),      # 48.2, 51.8
    (1024, 16384, 16, True, 3),     # 89.7, 86.8
    (1024, 4096, 32, True, 1),      # 28.6, 37.2
    (1024, 8192, 32, True, 3),      # 61.9, 59.1
    (1024, 64, 17, False, 2),       # 15.4, 11.5
    (900, 128, 32, False, 2),       # 14.3, 11.9
    (1025, 64, 4, True, 3), (64, 64, 33, True, 3)])
def test_projection_backward(T, d, E, with_dx, launches):
    s = B.make_shape(T, d, 64, E, 1, 8, I.BF16, I.GELU)
    assert B.moe_gate_logits_bwd_launches(s, with_dx, 0.0) == launches
    assert B.moe_gate_logits_bwd_launches(s, with_dx, 0.01) == (3 if with_dx else 2)


@pytest.mark.parametrize("T,d,E,dtype,eps,chunks", [
    (4096, 512, 32, I.BF16, 0.0, 32),       # 16 chunks 12.7, 32 12.0
    (4096, 1024, 64, I.BF16, 0.0, 16),      # 13.8, 15.2 with 32
    (5003, 776, 4, I.BF16, 0.0, 40),        # 20 chunks 13.4, 40 12.6
    (6000, 1024, 32, I.BF16, 0.0, 24),      # 14.0, 14.4 with 47
    (7000, 776, 16, I.BF16, 0.0, 28),       # 13.9, 14.5 with 55
    (32768, 64, 32, I.BF16, 0.0, 128),      # 16.0, 19.2 with 256
    (6000, 1024, 16, I.BF16, 0.01, 47),     # 24 chunks 33.3, 47 25.6
    (32768, 64, 32, I.BF16, 0.01, 256),     # 128 chunks 36.7, 256 31.2
    (12288, 64, 16, I.F32, 0.0, 192),       # 48 chunks 18.3, 192 17.4
    (16384, 64, 4, I.F32, 0.0, 64),         # 18.8, 19.2 with 256
    (65536, 1024, 32, I.BF16, 0.0, 128)])   # the chip is full twice
def test_projection_backward_chunks(T, d, E, dtype, eps, chunks):
    s = B.make_shape(T, d, 64, E, 1, 8, dtype, I.GELU)
    assert B.moe_gate_logits_bwd_chunks(s, eps) == chunks
    # the workspace that the query asks for holds every chunk's partial sums, with jitter and without
    assert B.moe_workspace_bytes(s) >= max(B.moe_gate_logits_bwd_chunks(s, e) for e in (0.0, 0.01)) * d * E * 4


@pytest.mark.parametrize("T,d,E,k,dtype,launches", [
    (256, 64, 4, 1, I.F32, 1),
    (16384, 64, 32, 2, I.BF16, 1),      # one pass 11.2, two 11.6
    (24576, 128, 4, 2, I.BF16, 2),      # 16.8, 15.8
    (32768, 64, 32, 2, I.BF16, 2),      # 20.2, 18.2
    (32768, 512, 32, 2, I.BF16, 1),     # 30.9, 31.2
    (65536, 512, 32, 2, I.BF16, 2),     # 81.4, 74.4
    (65536, 512, 32, 2, I.F32, 1),      # the same
    (32768, 64, 16, 1, I.F32, 1),       # the same
    (65536, 128, 16, 1, I.BF16, 2),     # 28.2, 25.7
    (65536, 64, 64, 1, I.F32, 1),       # 4 % faster in one
    (131072, 128, 256, 2, I.BF16, 1),   # 6 % faster in one
    (65536, 2048, 16, 2, I.BF16, 1)])
def test_combine_and_gate_backward(T, d, E, k, dtype, launches):
    assert B.moe_combine_gate_bwd_launches(B.make_shape(T, d, 64, E, k, max(1, T * k // E), dtype, I.GELU)) == launches


@pytest.mark.parametrize("dtype,d", [(I.F32, 1 << 22), (I.F32, 1 << 23), (I.F32, 1 << 24), (I.BF16, 1 << 23), (I.BF16, 1 << 24)])
def test_projection_backward_chunks_of_very_wide_tokens_keep_32_bit_offsets(dtype, d):
    """A chunk's rows of x are addressed with 32-bit byte offsets up to 2 GiB; rounding its tokens up must not pass that."""
    for T in (1025, 4096, 5003):
        s = B.make_shape(T, d, 8, 2, 1, 1, dtype, I.GELU)
        for eps in (0.0, 0.01):
            chunks = B.moe_gate_logits_bwd_chunks(s, eps)
            # every chunk but the last is full, so no chunk holds fewer tokens than this
            tokens = -(-T // chunks)
            assert tokens * d * (4 if dtype == I.F32 else 2) < 1 << 31, (T, chunks)


@pytest.mark.parametrize("T,d,f,E,k,C,dtype,direct", [
    # xd W1, h W2, dz with dW2, dxd with dW1: do all tiles that there could be have a CU each and mostly hold rows
    (256, 64, 256, 4, 1, 64, I.F32, [True] * 4),                # the four launches 18.8 direct, 25 through a table
    (512, 512, 2048, 8, 1, 64, I.BF16, [True, True, False, False]),
    (61, 64, 200, 3, 2, 129, I.BF16, [False] * 4),              # mostly empty
    (372, 1216, 1192, 8, 2, 117, I.BF16, [False] * 4),          # 304 tiles: 24 direct, 19 walked with a Zipf gate
    (3279, 272, 704, 6, 2, 1093, I.BF16, [False, True, False, False]),     # 324 tiles: 13.4, 12.2 with a hot expert
    (1746, 368, 1136, 5, 2, 699, I.F32, [False, False, False, True]),      # h W2 44, 30 with one expert taking all
    (360, 2008, 6312, 6, 1, 75, I.BF16, [False] * 4),           # h W2 48, 37 with one expert taking all
    (700, 1288, 2056, 1, 1, 700, I.BF16, [True, True, True, False]),       # 363 tiles, three per CU: an expert that has all
    (15413, 200, 768, 1, 1, 19267, I.BF16, [False, False, False, False]),  # h W2 16.5, 12.4: a fifth of 302 tiles is empty
])
def test_tiles_found_without_the_counts(T, d, f, E, k, C, dtype, direct):
    assert B.moe_expert_ffn_direct(B.make_shape(T, d, f, E, k, C, dtype, I.GELU)) == direct


@pytest.mark.parametrize("T,d,f,E,k,C,dtype", [
    (521, 96, 384, 19, 2, 55, I.F32),       # dxd with dW1, 114 + 684 tiles of 32 x 32: 800 workgroups 17.2 us, 808 8.2
    (6044, 88, 88, 5, 1, 1209, I.F32),      # both launches, 570 + 45: 616 16.6, 624 12.9
    (316, 352, 1408, 4, 2, 198, I.BF16),    # dxd with dW1, 96 + 528 of 64 x 64
    (1216, 96, 448, 29, 1, 84, I.BF16),
])
def test_a_round_of_both_products_has_whole_eighths_of_each(T, d, f, E, k, C, dtype):
    s = B.make_shape(T, d, f, E, k, C, dtype, I.GELU)
    up = lambda a, b: -(-a // b)
    for i, (N, M2, N2) in ((2, (f, f, d)), (3, (d, d, f))):
        side, groups = B.moe_expert_ffn_tiles(s)[i]
        first, second = E * up(C, side) * up(N, side), E * up(M2, side) * up(N2, side)
        most = 32 * (8 if side == 32 else {(I.BF16, 64): 3, (I.BF16, 128): 2, (I.F32, 64): 1, (I.F32, 128): 3 - groups}[dtype, side])
        assert side < 256 and B.moe_expert_ffn_workgroups(s)[i] == 8 * min(most, up(first, 8) + up(second, 8))


@pytest.mark.parametrize("rows,d,f,E,parts", [
    # fp32, few tiles: 32 x 32 in xd W1, h W2, dz with dW2, dxd with dW1
    (64, 64, 256, 4, [True] * 4),               # 5, 5, 5, 6; 64 x 64: 7, 8, 8, 9
    (311, 136, 328, 5, [True] * 4),             # one hot expert 7.8, 5.8, 10.8, 8.9; 9.2, 9.8, 11.8, 11.6
    (1675, 48, 96, 3, [True] * 4),              # long reductions over the rows, Zipf gate 7.0, 4.4, 17.5, 19.0; 7.7, 5.9, 33.6, 34.2
    (464, 176, 704, 3, [True] * 4),             # 12.0, 13.2, 16.6, 16.6; 14.9, 21.5, 18.7, 13.4
    (624, 192, 192, 8, [False, False, True, True]),     # full in one round of 64 x 64: 12.7, 10.6, 17.3, 17.2; 9.6, 6.8, 21.4, 20.2
    (461, 512, 512, 2, [True, True, False, False]),     # 18.2, 17.4; 13.1, 12.3 in the last two
    (300, 232, 232, 10, [False] * 4),
])
def test_fp32_tiles_of_small_products(rows, d, f, E, parts):
    s = B.make_shape(E * rows, d, f, E, 1, rows, I.F32, I.GELU)
    assert B.moe_expert_ffn_parts(s) == parts
    # and the query of the tiles names the kernel that runs: four waves on 32 x 32, two groups of four on 64 x 64
    assert B.moe_expert_ffn_tiles(s) == [(32, 1) if p else (64, 2) for p in parts]


def test_long_reductions_keep_64_x_64_tiles():
    # h W2 of 12 experts of 85 rows, K = 3864: 64 x 64 138, 32 x 32 159; 32 of 86, K = 2128: 81, 84 (82, 97 with a Zipf gate)
    for rows, d, f, E in ((85, 1288, 3864, 12), (86, 512, 2128, 32)):
        s = B.make_shape(E * rows, d, f, E, 1, rows, I.F32, I.GELU)
        assert B.moe_expert_ffn_tiles(s)[1] == (64, 2) and not B.moe_expert_ffn_parts(s)[1]


@pytest.mark.parametrize("rows,d,f,E,first,second", [
    # bf16, experts of at most 128 rows: tile side of dz with dW2 and of dxd with dW1
    (66, 864, 2256, 36, 128, 256),      # 90 with 128 x 128 against 127
    (74, 1200, 600, 24, 128, 128),      # 25, 49; 26, 36: the shorter extent is the other one
    (61, 1512, 1512, 6, 128, 128),      # 28, 42; 27, 36
    (46, 1512, 1512, 64, 128, 256),     # 238, 243; 235, 206
    (102, 1016, 1016, 100, 128, 256),   # 212, 206; 206, 181
    (74, 1992, 1528, 24, 128, 256),     # 139, 142; 126, 118
    (101, 968, 3840, 4, 128, 128),      # 26, 37; 42, 70
    (17, 1376, 2056, 12, 128, 128),     # 59, 74; 70, 79
    (66, 560, 1776, 100, 128, 128),     # 161, 160; 150, 202: fewer rounds
    (129, 1512, 1512, 64, 256, 256),
])
def test_backward_tiles_of_few_rows(rows, d, f, E, first, second):
    s = B.make_shape(E * rows, d, f, E, 1, rows, I.BF16, I.GELU)
    assert [t[0] for t in B.moe_expert_ffn_tiles(s)[2:]] == [first, second]
