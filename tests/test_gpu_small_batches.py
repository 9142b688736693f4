"""GPU: what small batches and the layer's fused calls run on - routing in one workgroup, the projection's backward in
one launch, combine and gate backward in one pass - at the edges of their ranges, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
import gpu_util as G

pytestmark = pytest.mark.gpu


def i32(*shape):
    return torch.full(shape, -7, dtype=torch.int32, device="cuda")


def f32(*shape):
    return torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("T,E,k,C,keys", [
    (1, 2, 2, 1, "uniform"), (63, 4, 1, 20, "ties"), (64, 3, 2, 50, "uniform"), (65, 5, 1, 9, "signed"),
    (256, 8, 2, 64, "ties"), (257, 130, 2, 3, "uniform"), (512, 64, 1, 8, None), (1000, 31, 2, 70, "signed"),
    (1023, 9, 2, 500, None), (1024, 32, 2, 64, "uniform"), (1024, 1, 1, 1000, "ties"),
    (1025, 32, 2, 64, "uniform"), (200, 256, 1, 200, "uniform"),        # beyond one workgroup's range, as are some above
    # the largest batches that one workgroup takes, per number of lanes that share a token
    (384, 32, 2, 24, "ties"), (384, 32, 1, 12, None), (768, 16, 2, 90, "signed"), (900, 16, 1, 56, None),
    (1024, 8, 1, 2048, "signed"), (1024, 4, 2, 4096, "ties"), (96, 64, 2, 40, "ties"), (64, 128, 1, 20, "signed"),
    (32, 256, 2, 3, "uniform"), (20, 130, 2, 1, None)])
def test_route_small(T, E, k, C, keys):
    rng = np.random.default_rng(T * 7 + E)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    lg[rng.random(T) < 0.2, :min(2, E)] = 1.5                           # tied logits
    kv = {None: None, "uniform": rng.random(T, dtype=np.float32),
          "ties": rng.integers(0, 4, T).astype(np.float32) / 4,
          "signed": np.where(rng.random(T) < 0.3, rng.choice([0.0, -0.0], T), rng.standard_normal(T) * 1e3).astype(np.float32)}[keys]
    s = B.make_shape(T, 8, 8, E, k, C, I.F32, I.GELU)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    probs, gw, ei, slot, cnt, dem, src = f32(T, E), f32(T, k), i32(T, k), i32(T, k), i32(E), i32(E), i32(E, C)
    util = torch.zeros(E, dtype=torch.int64, device="cuda")
    lgd, kd = G.to_dev(lg, I.F32), G.to_dev(kv, I.F32)
    print(f"[gpu] route T={T} E={E} k={k} C={C} keys={keys}", flush=True)
    for _ in range(2):
        B.moe_gate_route_counted(s, 1, lgd, kd, probs, ei, gw, slot, cnt, dem, src, util, ws)
    torch.cuda.synchronize()
    p = O.softmax(lg)
    idx = O.top_k(lg, k)
    rslot, rcnt, rdem, rsrc = O.route(idx, kv, E, C)
    for name, got, want in (("expert_idx", ei, idx), ("slot", slot, rslot), ("count", cnt, rcnt), ("demand", dem, rdem),
                            ("slot_src", src, rsrc), ("utilisation", util, 2 * rdem.astype(np.int64))):
        assert np.array_equal(got.cpu().numpy(), want), name
    assert G.rel_l2(G.host(probs), p) <= 1e-5
    assert G.rel_l2(G.host(gw), O.gate_weights(p, idx)) <= 1e-5


@pytest.mark.parametrize("dtype", [I.F32, I.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("T,d,E,k,aux", [(1, 8, 2, 2, 0.0), (130, 72, 5, 2, 0.0), (777, 520, 32, 1, 0.01),
                                         (300, 1032, 130, 2, 0.01), (515, 64, 256, 2, 0.0), (64, 8, 1, 1, 0.01),
                                         # two passes: many tokens of short rows
                                         (24577, 72, 6, 2, 0.0), (24577, 72, 6, 2, 0.01), (49153, 72, 7, 1, 0.0)])
def test_combine_and_gate_backward(T, d, E, k, aux, dtype):
    rng = np.random.default_rng(T + E)
    C = max(1, (T * k) // E)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    p, idx = O.softmax(lg), O.top_k(lg, k)
    gw = O.gate_weights(p, idx).astype(np.float32)
    slot, cnt, _, _ = O.route(idx, rng.random(T, dtype=np.float32), E, C)
    dy = rng.standard_normal((T, d)).astype(np.float32)
    yd = rng.standard_normal((E, C, d)).astype(np.float32)
    if dtype == I.BF16:
        dy, yd = I.round_to_bf16(dy), I.round_to_bf16(yd)
    s = B.make_shape(T, d, 8, E, k, C, dtype, I.GELU)
    dyd = torch.zeros((E, C, d), dtype=torch.bfloat16 if dtype == I.BF16 else torch.float32, device="cuda")
    dg, dl = f32(T, k), f32(T, E)
    p32 = p.astype(np.float32)
    ff = O.aux_loss(p, idx)[1].astype(np.float32) if aux else None
    print(f"[gpu] combine + gate backward T={T} d={d} E={E} k={k} aux={aux}", flush=True)
    B.moe_combine_gate_bwd(s, G.to_dev(dy, dtype), G.to_dev(yd, dtype), G.to_dev(idx.astype(np.int32), None),
                           G.to_dev(slot, None), G.to_dev(gw, I.F32), G.to_dev(p32, I.F32), G.to_dev(ff, I.F32), aux,
                           dyd, dg, dl)
    torch.cuda.synchronize()
    rdyd, rdg = O.combine_bwd(dy, yd, idx, slot, gw)
    rdl = O.gate_bwd(rdg, p32, idx, slot)
    if aux:
        rdl = rdl + O.aux_loss_bwd(p32, ff, aux)
    m = G.row_mask(cnt, C)
    assert G.rel_l2(G.host(dyd)[m], rdyd[m]) <= G.TOL[dtype]
    # dlogits in place of the probabilities
    pd, dg2 = G.to_dev(p32, I.F32), f32(T, k)
    B.moe_combine_gate_bwd(s, G.to_dev(dy, dtype), G.to_dev(yd, dtype), G.to_dev(idx.astype(np.int32), None),
                           G.to_dev(slot, None), G.to_dev(gw, I.F32), pd, G.to_dev(ff, I.F32), aux, dyd, dg2, pd)
    torch.cuda.synchronize()
    assert G.rel_l2(G.host(pd), rdl) <= 1e-5
    # fp32 sums of products of given values, whatever the activation type
    assert G.rel_l2(G.host(dg), rdg) <= 1e-5
    assert G.rel_l2(G.host(dl), rdl) <= 1e-5


@pytest.mark.parametrize("dtype", [I.F32, I.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("T,d,E,with_dx", [(1, 8, 1, True), (31, 24, 3, True), (33, 136, 4, False), (255, 520, 8, True),
                                           (513, 72, 9, True), (600, 136, 17, True), (1024, 264, 32, True),
                                           (1025, 72, 32, True),        # three launches
                                           (512, 72, 32, False), (1024, 72, 16, False),     # one, without dx
                                           (513, 72, 17, False), (700, 4104, 17, True), (7, 12296, 4, True)])   # beyond the line
def test_projection_backward_small(T, d, E, with_dx, dtype):
    rng = np.random.default_rng(T + d + E)
    x, dx0 = rng.standard_normal((T, d)).astype(np.float32), rng.standard_normal((T, d)).astype(np.float32)
    if dtype == I.BF16:
        x, dx0 = I.round_to_bf16(x), I.round_to_bf16(dx0)
    Wg, dl = rng.standard_normal((d, E)).astype(np.float32), rng.standard_normal((T, E)).astype(np.float32)
    s = B.make_shape(T, d, 8, E, 1, 4, dtype, I.GELU)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    dWg, dx = f32(d, E), G.to_dev(dx0, dtype)
    print(f"[gpu] projection backward T={T} d={d} E={E}", flush=True)
    B.moe_gate_logits_bwd(s, G.to_dev(x, dtype), G.to_dev(Wg, I.F32), G.to_dev(dl, I.F32), dWg, dx if with_dx else None, ws)
    torch.cuda.synchronize()
    rdWg, rdx = O.gate_logits_bwd(x, Wg, dl)
    assert G.rel_l2(G.host(dWg), rdWg) <= 1e-5
    assert G.rel_l2(G.host(dx), dx0 + (rdx if with_dx else 0.0)) <= G.TOL[dtype]


@pytest.mark.parametrize("dtype", [I.F32, I.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("eps", [0.0, 0.01], ids=["plain", "jitter"])
@pytest.mark.parametrize("T,d,E", [(1025, 72, 5), (1153, 264, 33), (2049, 520, 8), (4100, 264, 16)])
def test_projection_backward_short_chunks(T, d, E, eps, dtype):
    """Token chunks of one or two rounds, the last one with a few tokens."""
    rng = np.random.default_rng(T + d)
    x = rng.standard_normal((T, d)).astype(np.float32)
    if dtype == I.BF16:
        x = I.round_to_bf16(x)
    Wg, dl = rng.standard_normal((d, E)).astype(np.float32), rng.standard_normal((T, E)).astype(np.float32)
    s = B.make_shape(T, d, 8, E, 1, 4, dtype, I.GELU)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    dWg = f32(d, E)
    print(f"[gpu] projection backward T={T} d={d} E={E} eps={eps}", flush=True)
    B.moe_gate_logits_bwd_jitter(s, G.to_dev(x, dtype), G.to_dev(Wg, I.F32), G.to_dev(dl, I.F32), eps, 11, dWg, None, ws)
    torch.cuda.synchronize()
    noise = O.jitter_noise(T, d, eps, 11) if eps else 1.0
    # fp32 sums of T products: the same bound as the other projection tests
    assert G.rel_l2(G.host(dWg), O.gate_logits_bwd(x * noise, Wg, dl)[0]) <= 1e-5


@pytest.mark.parametrize("groups,chunks,E,k", [(2, 1, 3, 2), (17, 1, 8, 1), (3, 5, 130, 2), (5, 7, 16, 2), (2, 16, 200, 1),
                                               (3, 16, 9, 2), (2, 32, 5, 1), (6, 17, 4, 1)])
def test_route_grouped_offsets(groups, chunks, E, k):
    """Rows kept by earlier groups, from histogram runs that end inside, at and beyond a batch of loads."""
    T = groups * chunks * 256
    C = groups * max(1, T * k // (2 * E * groups))                      # half the demand fits
    rng = np.random.default_rng(groups * 100 + chunks)
    lg = (rng.standard_normal((T, E)) + np.linspace(0.0, 2.0, E)).astype(np.float32)
    keys = rng.random(T, dtype=np.float32)
    s = B.make_shape(T, 8, 8, E, k, C, I.F32, I.GELU)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    probs, gw, ei, slot, cnt, dem, src = f32(T, E), f32(T, k), i32(T, k), i32(T, k), i32(E), i32(E), i32(E, C)
    print(f"[gpu] grouped route T={T} groups={groups} E={E} k={k}", flush=True)
    B.moe_gate_route_grouped(s, groups, G.to_dev(lg, I.F32), G.to_dev(keys, I.F32), probs, ei, gw, slot, cnt, dem, src, ws)
    torch.cuda.synchronize()
    idx = O.top_k(lg, k)
    rslot, rcnt, rdem, rsrc = O.route_grouped(idx, keys, E, C, groups)
    for name, got, want in (("expert_idx", ei, idx), ("slot", slot, rslot), ("count", cnt, rcnt), ("demand", dem, rdem),
                            ("slot_src", src, rsrc)):
        assert np.array_equal(got.cpu().numpy(), want), name


@pytest.mark.parametrize("T,d,E", [(1, 8, 1), (31, 72, 3), (33, 512, 8), (33, 520, 8), (65, 1032, 31), (8192, 520, 5), (8193, 520, 5)])
def test_gate_projection_tiles(T, d, E):
    """One and two token tiles per workgroup, at the lines between them."""
    rng = np.random.default_rng(T + d)
    x, Wg = I.round_to_bf16(rng.standard_normal((T, d)).astype(np.float32)), rng.standard_normal((d, E)).astype(np.float32)
    logits = f32(T, E)
    print(f"[gpu] gate projection T={T} d={d} E={E}", flush=True)
    B.moe_gate_logits(B.make_shape(T, d, 8, E, 1, 4, I.BF16, I.GELU), G.to_dev(x, I.BF16), G.to_dev(Wg, I.F32), None, logits)
    torch.cuda.synchronize()
    assert G.rel_l2(G.host(logits), O.gate_logits(x, Wg, None)) <= 1e-5     # fp32 sums of products that the split leaves exact


@pytest.mark.parametrize("dtype", [I.F32, I.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("T,d,E", [(64, 72, 4), (700, 264, 8), (1024, 1032, 30)])
def test_projection_backward_in_place_of_its_tokens(T, d, E, dtype):
    """dx written over x: dWg is that of the tokens as they were, whatever the number of launches."""
    rng = np.random.default_rng(T)
    x = rng.standard_normal((T, d)).astype(np.float32)
    if dtype == I.BF16:
        x = I.round_to_bf16(x)
    Wg, dl = rng.standard_normal((d, E)).astype(np.float32), rng.standard_normal((T, E)).astype(np.float32)
    s = B.make_shape(T, d, 8, E, 1, 4, dtype, I.GELU)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    xd, dWg = G.to_dev(x, dtype), f32(d, E)
    print(f"[gpu] projection backward in place T={T} d={d} E={E}", flush=True)
    B.moe_gate_logits_bwd(s, xd, G.to_dev(Wg, I.F32), G.to_dev(dl, I.F32), dWg, xd, ws)
    torch.cuda.synchronize()
    rdWg, rdx = O.gate_logits_bwd(x, Wg, dl)
    assert G.rel_l2(G.host(dWg), rdWg) <= 1e-5
    assert G.rel_l2(G.host(xd), x + rdx) <= G.TOL[dtype]
