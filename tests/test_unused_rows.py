"""Rows from expert_count[e] on of the per-expert buffers are never read and never written, whatever finds a tile's rows."""
import os
import re

import numpy as np
import pytest
import torch

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

CSRC = os.path.join(os.path.dirname(os.path.abspath(B.__file__)), "csrc")


def test_every_bound_of_the_row_operand_is_the_rows_in_use():
    """A read of an unused row changes no result (it meets only outputs that are not stored), so no run can show it.  What
    decides it is the bound that each kernel gives to its operand A: in the source it must be the walk's row limit."""
    src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "expert_gemm.hip")).read())
    kernels = src[src.index("gemm_body(const GemmArgs& p"):src.index("static int num_cus()")]
    bounds = re.findall(r"TA::(?:plan|desc)\(([^;]*)\);", kernels)                              # bf16
    bounds += re.findall(r"rangeA = ([^;]*);", kernels)                                         # fp32 through LDS
    bounds += re.findall(r"rsA = buf_rsrc\(\(const float\*\)[pq]\.A([^;]*)\);", kernels)        # fp32 from memory
    assert len(bounds) == 7, bounds
    for b in bounds:
        assert re.search(r"\b(?:p?w\.)?m_lim\b", b), b


# buffers that are mostly full (a workgroup of the small tiles may find its tile before it knows the row count) and
# half-empty ones; tile (side, wave groups) of xd W1, h W2, dz with dW2, dxd with dW1
#        name            E    C     d     f  rows expected  dtype
SHAPES = [
    ("f32_small",        4,   40,   72,  136,    40, I.F32),
    ("f32_few_columns",  8,  624,  192,  192,   624, I.F32),
    ("f32_128_groups",   8,  380,  136, 1032,   380, I.F32),
    ("f32_one_expert",   1, 1219,  840,  840,  1219, I.F32),
    ("f32_half_empty",   5,  240,   72,  136,   120, I.F32),
    ("f32_65_experts",  65,   40,   24,   40,    40, I.F32),
    ("bf16_64",          4,   40,   72,  136,    40, I.BF16),
    ("bf16_128",         8,  300,  520, 1032,   300, I.BF16),
    ("bf16_one_expert",  1,  700, 1288, 2056,   700, I.BF16),
    ("bf16_half_empty",  8,  300,  520, 1032,   150, I.BF16),
    ("bf16_65_experts", 65,   40,   72,  136,    40, I.BF16),
    ("bf16_256",         8,  700,  520, 2056,   700, I.BF16),
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,E,C,d,f,rows,dtype", SHAPES, ids=[s[0] for s in SHAPES])
def test_what_lies_behind_the_rows_in_use_does_not_matter(name, E, C, d, f, rows, dtype):
    """NaN and infinities there neither change a result nor are written over."""
    s = B.make_shape(E * rows, d, f, E, 1, C, dtype, I.GELU)
    rng = np.random.default_rng(7)
    cnt = np.minimum(rng.integers(rows - rows // 8, rows + 1, E), C).astype(np.int32)
    cnt[0] = max(1, rows - 7)
    if E > 2:
        cnt[1], cnt[2] = 1, 0
    tdt = torch.bfloat16 if dtype == I.BF16 else torch.float32
    dev = lambda *sh: torch.from_numpy(rng.standard_normal(sh, dtype=np.float32)).cuda().to(tdt)
    xd, dyd, W1, W2 = dev(E, C, d), dev(E, C, d), 0.1 * dev(E, d, f), 0.1 * dev(E, f, d)
    unused = torch.arange(C, device="cuda")[None, :] >= torch.from_numpy(cnt).cuda()[:, None]
    c = G.to_dev(cnt, None)
    ref = None
    for fill in (0.0, float("nan"), float("inf")):
        xd[unused], dyd[unused] = fill, fill
        new = lambda m: torch.full((E, C, m), fill, device="cuda", dtype=tdt)
        h, a, yd, dxd, he, ye = new(f), new(f), new(d), new(d), new(f), new(d)
        dW1, dW2 = torch.full((E, d, f), fill, device="cuda"), torch.full((E, f, d), fill, device="cuda")
        ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
        ws[:ws.numel() // 4 * 4].view(torch.float32).fill_(fill)
        print(f"[gpu] {name}: unused rows hold {fill}", flush=True)
        B.moe_expert_ffn_fwd(s, xd, c, W1, W2, h, a, yd)
        B.moe_expert_ffn_fwd(s, xd, c, W1, W2, he, None, ye)
        B.moe_expert_ffn_bwd(s, dyd, xd, h, a, c, W1, W2, dxd, dW1, dW2, ws)
        torch.cuda.synchronize()
        for t in (h, a, yd, dxd, he, ye):
            assert bool((t[unused].isnan() if fill != fill else t[unused] == fill).all())
        got = [t[~unused].float() for t in (h, a, yd, dxd, he, ye)] + [dW1, dW2]
        assert all(bool(t.isfinite().all()) for t in got)
        if ref is None:
            ref = got
        assert all(torch.equal(x, y) for x, y in zip(ref, got))
