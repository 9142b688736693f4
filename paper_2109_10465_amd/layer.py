"""Buffer owner and call sequence for one MoE layer step on one GPU.

Holds the device buffers (torch tensors used as raw memory) and makes the two
C-ABI calls of a step: moe_layer_fwd (gate -> capacity/RTS -> dispatch -> experts
-> combine) and moe_layer_bwd, its reverse.  No arithmetic happens here.
"""
import torch

from . import binding as B

_TORCH_DT = {B.F32: torch.float32, B.BF16: torch.bfloat16}


class MoELayer:
    def __init__(self, T, d_model, d_ff, E, k, capacity, dtype, act, device="cuda:0", aux_coef=0.0,
                 forward_only=False, groups=1, jitter_eps=0.0, drop_p=0.0):
        if not torch.cuda.is_available():
            raise B.MoeError("MoELayer needs a GPU; there is no CPU fallback")
        B.lib()
        self.shape = B.make_shape(T, d_model, d_ff, E, k, capacity, dtype, act)
        self.T, self.d, self.f, self.E, self.k, self.C = T, d_model, d_ff, E, k, capacity
        self.device = torch.device(device)
        self.aux_coef = float(aux_coef)     # weight of the balancing loss in the objective (0 = off)
        self.jitter_eps = float(jitter_eps)  # gate jitter (training); the seed is given per step
        self.drop_p = float(drop_p)          # expert dropout on the hidden activation (training)
        self.seed = 0
        self.groups = int(groups)           # > 1: token selection inside groups of T/groups consecutive tokens
        self.forward_only = bool(forward_only)   # evaluation: no saved derivative, no backward buffers
        adt = _TORCH_DT[dtype]
        dev = self.device

        def buf(shape, dt):
            return torch.empty(shape, dtype=dt, device=dev)

        i32, f32 = torch.int32, torch.float32
        self.logits = buf((T, E), f32)
        self.probs = buf((T, E), f32)
        self.expert_idx = buf((T, k), i32)
        self.gate_w = buf((T, k), f32)
        self.slot = buf((T, k), i32)
        self.expert_count = buf((E,), i32)
        self.expert_demand = buf((E,), i32)
        self.slot_src = buf((E, capacity), i32)
        self.first_frac = buf((E,), f32)     # balancing loss: first-choice share, mean probability, value
        self.mean_prob = buf((E,), f32)
        self.aux_loss = buf((1,), f32)
        self.xd = buf((E, capacity, d_model), adt)
        self.h = buf((E, capacity, d_ff), adt)       # act(z)
        self.dact = None if forward_only else buf((E, capacity, d_ff), adt)    # act'(z)
        self.yd = buf((E, capacity, d_model), adt)
        self.y = buf((T, d_model), adt)
        self.utilisation = torch.zeros((E,), dtype=torch.int64, device=dev)   # tokens routed to each expert so far
        nbytes = B.moe_workspace_bytes(self.shape)
        if nbytes == 0:
            raise B.MoeError("unsupported shape")
        self.ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        if forward_only:
            return
        # backward
        self.dyd = buf((E, capacity, d_model), adt)
        self.dgate_w = buf((T, k), f32)
        self.dxd = buf((E, capacity, d_model), adt)
        self.dW1 = buf((E, d_model, d_ff), f32)
        self.dW2 = buf((E, d_ff, d_model), f32)
        self.dlogits = buf((T, E), f32)
        self.dWg = buf((d_model, E), f32)
        self.dx = buf((T, d_model), adt)

    # what moe_layer_fwd and moe_layer_bwd take, in the order of B.LayerBuffers; a forward-only layer has no
    # derivative and no backward buffers
    _FWD = ("logits", "probs", "expert_idx", "gate_w", "slot", "expert_count", "expert_demand", "slot_src",
            "utilisation", "first_frac", "mean_prob", "aux_loss", "xd", "h", "dact", "yd", "y")
    _BWD = ("dyd", "dgate_w", "dxd", "dW1", "dW2", "dlogits", "dWg", "dx")

    def _call_args(self, logits_given=False):
        """Options and buffers of one call, from the layer's attributes as they are now."""
        at = self.__dict__
        ptrs = [None if at[n] is None else at[n].data_ptr() for n in self._FWD]
        ptrs += [None] * len(self._BWD) if self.forward_only else [None if at[n] is None else at[n].data_ptr() for n in self._BWD]
        # attributes may have been set anew since: whatever is a number, and fewer than two groups is plain routing
        return (B.LayerOptions(max(1, int(self.groups)), bool(self.forward_only), logits_given, self.aux_coef,
                               self.jitter_eps, self.drop_p, int(self.seed) & 0xFFFFFFFFFFFFFFFF),
                B.LayerBuffers(*ptrs, self.ws.data_ptr(), self.ws.numel() * self.ws.element_size()))

    def forward(self, x, Wg, bias, W1, W2, rts_keys, logits=None, seed=0):
        """logits: optional precomputed [T,E] fp32 gate logits; the projection call is
        then skipped and routing runs on exactly these values."""
        self._saved = (x, Wg, W1, W2)
        self.seed = int(seed)     # of this step's jitter and dropout draws
        if logits is not None:
            self.logits.copy_(logits)
        B.moe_layer_fwd(self.shape, *self._call_args(logits is not None), x, Wg, bias, W1, W2, rts_keys)
        return self.y

    def backward(self, dy):
        if self.forward_only:
            raise B.MoeError("this layer was built forward-only")
        x, Wg, W1, W2 = self._saved
        B.moe_layer_bwd(self.shape, *self._call_args(), x, Wg, W1, W2, dy)
        return self.dx, self.dWg, self.dW1, self.dW2

    def step(self, x, Wg, bias, W1, W2, rts_keys, dy, logits=None, seed=0):
        self.forward(x, Wg, bias, W1, W2, rts_keys, logits, seed)
        return self.backward(dy)

    def capture_step(self, x, Wg, bias, W1, W2, rts_keys, dy, seed=0):
        """Records one forward+backward step into a HIP graph and returns it (`.replay()` runs the step again on
        the same tensors: refill x, dy, the weights and the keys in place between replays).  The library
        allocates nothing and clears nothing with memset, so every call of the step is a plain kernel node.
        Replay takes the host out of the loop (18 us of host time instead of 44 for a 256-token step); the time of a
        step stays about the same, since the chain of dependent kernels sets it, not their launch (256 tokens, fp32:
        51 us eager; 55 eager and 57 replayed when its expert products took 1-2 us longer each).
        The seed of the step's noise draws is a host value and is recorded with the graph."""
        if self.forward_only:
            raise B.MoeError("this layer was built forward-only")
        self.step(x, Wg, bias, W1, W2, rts_keys, dy, seed=seed)       # first use of every kernel happens eagerly
        torch.cuda.synchronize(self.device)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            self.step(x, Wg, bias, W1, W2, rts_keys, dy, seed=seed)
        return graph
