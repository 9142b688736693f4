"""What MoELayer hands to the native calls, from attributes as a program may set them (no GPU: the layer's constructor,
which needs one, is passed by)."""
import numpy as np
import pytest
import torch

from paper_2109_10465_amd.layer import MoELayer


def layer(**over):
    m = object.__new__(MoELayer)
    for n in MoELayer._FWD + MoELayer._BWD:
        setattr(m, n, torch.zeros(4))
    m.ws = torch.zeros(1024, dtype=torch.uint8)
    m.groups, m.forward_only, m.aux_coef, m.jitter_eps, m.drop_p, m.seed = 1, False, 0.0, 0.0, 0.0, 0
    for n, v in over.items():
        setattr(m, n, v)
    return m


@pytest.mark.parametrize("groups,want", [(0, 1), (-3, 1), (1, 1), (8, 8), (np.int64(4), 4), (np.int32(0), 1)])
def test_groups(groups, want):
    assert layer(groups=groups)._call_args()[0].groups == want


def test_numbers_of_other_types():
    o = layer(forward_only=np.bool_(True), aux_coef=np.float32(0.5), jitter_eps=torch.tensor(0.25), drop_p=np.float64(0.125),
              seed=np.int64(-1))._call_args(True)[0]
    assert (o.forward_only, o.logits_given, o.aux_coef, o.jitter_eps, o.drop_p) == (1, 1, 0.5, 0.25, 0.125)
    assert o.seed == 2 ** 64 - 1


def test_workspace_is_given_in_bytes_and_missing_buffers_as_null():
    b = layer(ws=torch.zeros(256, dtype=torch.float32), dx=None, dact=None)._call_args()[1]
    assert b.ws_bytes == 1024 and b.dx is None and b.dact is None and b.dWg
