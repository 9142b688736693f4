"""The C-ABI library loads without a GPU, exports every symbol the header
declares, and its host-only entry points behave as documented.  No kernel is
launched here."""
import ctypes
import os
import re

import pytest

from oracle import moe_oracle as O
from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    """Every function declared in include/*.h (the layer's ABI and the measurement aid's header)."""
    names = set()
    inc = os.path.join(ROOT, "include")
    for fn in sorted(os.listdir(inc)):
        if fn.endswith(".h"):
            text = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, fn)).read(), flags=re.S)
            names |= set(re.findall(r"\b(moe_[a-z_0-9]+)\s*\(", text))
    return sorted(names)


def test_every_declared_symbol_is_exported_and_bound():
    names = declared_symbols()
    assert len(names) >= 14
    L = B.lib()
    for n in names:
        assert hasattr(L, n), n
    assert sorted(B.EXPORTS) == names
    for n in names:
        assert callable(getattr(B, n))


def test_capacity_rule_matches_oracle_and_workloads():
    for w in I.WORKLOADS.values():
        assert B.moe_capacity(w.T, w.E, w.k, w.capacity_factor) == w.capacity
    for T, E, k, cf in [(10, 4, 1, 1.0), (1, 64, 1, 1.0), (100, 8, 2, 2.0), (4096, 8, 2, 1.25),
                        (777, 5, 2, 1.1), (33, 7, 1, 0.5)]:
        assert B.moe_capacity(T, E, k, cf) == O.capacity(T, E, k, cf)
    assert B.moe_capacity(0, 4, 1, 1.0) == -1
    assert B.moe_capacity(16, 4, 3, 1.0) == -1
    assert B.moe_capacity(16, 4, 1, -1.0) == -1


def test_workspace_query_and_shape_validation():
    for w in I.WORKLOADS.values():
        s = B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.capacity, w.dtype, w.act)
        n = B.moe_workspace_bytes(s)
        assert n > 0 and n % 256 == 0
        # at least the backward's dz buffer
        assert n >= w.E * w.capacity * w.d_ff * (2 if w.dtype == I.BF16 else 4)
    bad = [
        B.make_shape(64, 12, 16, 4, 1, 16, 0, 0),     # d_model % 8
        B.make_shape(64, 16, 16, 4, 3, 16, 0, 0),     # k
        B.make_shape(64, 16, 16, 1, 2, 16, 0, 0),     # E < k
        B.make_shape(64, 16, 16, 300, 1, 16, 0, 0),   # E > 256
        B.make_shape(0, 16, 16, 4, 1, 16, 0, 0),      # T
        B.make_shape(64, 16, 16, 4, 1, 0, 0, 0),      # capacity
        B.make_shape(64, 16, 16, 4, 1, 16, 5, 0),     # dtype
        B.make_shape(64, 16, 16, 4, 1, 16, 0, 9),     # act
    ]
    for s in bad:
        assert B.moe_workspace_bytes(s) == 0


def test_argument_errors_are_reported_before_any_launch():
    # invalid shapes / NULL pointers return an error code on the host; nothing
    # touches a device, so this runs without one
    L = B.lib()
    bad = B.make_shape(64, 12, 16, 4, 1, 16, 0, 0)
    assert L.moe_gate_logits(ctypes.byref(bad), None, None, None, None, None) == -2
    ok = B.make_shape(64, 16, 16, 4, 1, 16, 0, 0)
    assert L.moe_gate_logits(ctypes.byref(ok), None, None, None, None, None) == -1
    assert L.moe_dispatch(ctypes.byref(ok), None, None, None, None, None) == -1
    assert L.moe_gate_bwd(None, None, None, None, None, None, None) == -1
    baddt = B.make_shape(64, 16, 16, 4, 1, 16, 7, 0)
    assert L.moe_combine_fwd(ctypes.byref(baddt), None, None, None, None, None, None) == -3
    assert B.moe_status_string(0) == "ok"
    assert "workspace" in B.moe_status_string(-4)
    with pytest.raises(B.MoeError):
        B._check(-2, "x")


LAYER_FWD = ("logits", "probs", "expert_idx", "gate_w", "slot", "expert_count", "expert_demand", "slot_src", "xd", "h", "yd", "y")
LAYER_BWD = ("probs", "expert_idx", "gate_w", "slot", "expert_count", "xd", "h", "dact", "yd", "dyd", "dgate_w", "dxd", "dW1",
             "dW2", "dlogits", "dWg", "dx")


def layer_call(backward, shape=(64, 16, 16, 4, 1, 16, 0, 0), without=(), inputs=(1, 1, 1, 1, 1), ws=None, **options):
    """The native layer call on buffers that are never touched (each "pointer" is just not NULL): what it returns is the
    host's verdict on the arguments."""
    s = B.make_shape(*shape)
    somewhere = 1 << 20
    buffers = B.LayerBuffers()
    for n, _ in B.LayerBuffers._fields_:
        setattr(buffers, n, None if n in without else somewhere)
    buffers.ws_bytes = B.moe_workspace_bytes(s) if ws is None else ws
    o = B.LayerOptions(groups=1)
    for n, v in options.items():
        setattr(o, n, v)
    x, Wg, W1, W2, dy = (somewhere if i else None for i in inputs)
    L = B.lib()
    if backward:
        return L.moe_layer_bwd(ctypes.byref(s), ctypes.byref(o), ctypes.byref(buffers), x, Wg, W1, W2, dy, None)
    return L.moe_layer_fwd(ctypes.byref(s), ctypes.byref(o), ctypes.byref(buffers), x, Wg, None, W1, W2, None, None)


def test_layer_calls_report_every_argument_error_before_their_first_launch():
    """An error of a late step of the pass comes back as that step's code.  Had an earlier step been issued by then, this
    process, which has no device, would get MOE_ERR_LAUNCH from it."""
    L = B.lib()
    s, o, b = B.make_shape(64, 16, 16, 4, 1, 16, 0, 0), B.LayerOptions(groups=1), B.LayerBuffers()
    for args in ((None, o, b), (s, None, b), (s, o, None)):
        args = [a if a is None else ctypes.byref(a) for a in args]
        assert L.moe_layer_fwd(*args, *[None] * 7) == -1
        assert L.moe_layer_bwd(*args, *[None] * 6) == -1
    for name in LAYER_FWD:
        assert layer_call(False, without=(name,)) == -1, name
    for name in LAYER_BWD:
        assert layer_call(True, without=(name,)) == -1, name
    for i in range(4):
        assert layer_call(False, inputs=[j != i for j in range(5)]) == -1, i
    for i in range(5):
        assert layer_call(True, inputs=[j != i for j in range(5)]) == -1, i
    assert layer_call(False, without=("utilisation",), forward_only=1) == -1
    for name in ("first_frac", "mean_prob", "aux_loss"):
        assert layer_call(False, without=(name,), aux_coef=0.01) == -1, name
    assert layer_call(True, without=("first_frac",), aux_coef=0.01) == -1
    assert layer_call(False, without=("dact",), drop_p=0.4) == -1
    big = (64, 1 << 16, 1 << 14, 4, 1, 16, 0, 0)            # beyond the expert FFN's slice limits
    small = (64, 16, 16, 4, 1, 16, 0, 0)
    for backward in (False, True):
        assert layer_call(backward, groups=0) == -2
        assert layer_call(backward, jitter_eps=1.5) == -2
        assert layer_call(backward, shape=big) == -2
        assert layer_call(backward, ws=16) == -4
        assert layer_call(backward, without=("ws",)) == -4
    assert layer_call(False, shape=small, groups=3) == -2   # 64 tokens are no three groups of whole chunks
    assert layer_call(False, drop_p=1.0) == -2
    wide = (64, 512, 8, 32, 1, 1, 0, 0)
    assert layer_call(True, shape=wide, ws=32 * 8 * 4) == -4        # enough for the experts' backward, not for the projection's


def test_build_rejects_scratch_in_kernels_with_hand_issued_loads():
    """A kernel that issues loads through inline asm and waits for them by hand must not spill: the build reads the
    compiler's resource-usage remarks and fails if such a kernel reports scratch memory."""
    from paper_2109_10465_amd import build as bld
    remark = ("gate.hip:1:1: remark: Function Name: _Z22gate_logits_lds_kernelILi4EEviiiPKtPKfS3_Pf [-Rpass-analysis]\n"
              "gate.hip:1:1: remark:     VGPRs: 168 [-Rpass-analysis]\n"
              "gate.hip:1:1: remark:     ScratchSize [bytes/lane]: {n} [-Rpass-analysis]\n")
    bld.check_no_scratch("gate.hip", remark.format(n=0))
    with pytest.raises(RuntimeError):
        bld.check_no_scratch("gate.hip", remark.format(n=28))
    # other kernels of the same file may spill
    bld.check_no_scratch("gate.hip", remark.format(n=28).replace("gate_logits_lds_kernel", "gate_dx_kernel"))


def test_static_routing_scratch_holds_the_shape_the_header_names():
    """moe_hip.h promises that the built-in scratch of moe_gate_route_static is enough for T = 65536, k = 2 with any
    E <= 256.  With tiny d_model, d_ff and capacity the routing workspace is the largest one, so the general
    workspace size is the routing workspace size (host-only calls)."""
    B.lib()
    cap = B.moe_gate_route_static_max_bytes()
    for E in (2, 32, 64, 65, 128, 129, 256):
        s = B.make_shape(65536, 8, 8, E, 2, 1, 0, 0)
        assert 0 < B.moe_workspace_bytes(s) <= cap, E
    assert B.moe_workspace_bytes(B.make_shape(1 << 21, 8, 8, 256, 2, 1, 0, 0)) > cap
