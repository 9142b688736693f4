// moe_layer_fwd / moe_layer_bwd: the entry points of one layer pass in order (host code only).  A call
// through a foreign-function interface costs several times what issuing a launch does; a 256-token step
// is ten launches of 2 to 9 us: with eight calls the host needed 70 us for it and set its time, with these two
// 44 of the 51 us that the step takes (43 on a faster host).
#include "moe_common.h"

static int check_args(const moe_shape* s, const moe_layer_options* o, const moe_layer_buffers* b) {
    if (!s || !o || !b) return MOE_ERR_NULL;
    return o->groups >= 1 ? MOE_OK : MOE_ERR_SHAPE;
}

// Everything that a step of the pass could refuse is checked before the first one is issued: an error leaves all
// outputs as they were (the utilisation count among them, which a second try would add to again).
static int check_fwd(const moe_shape* s, const moe_layer_options* o, const moe_layer_buffers* b, const void* x,
                     const float* Wg, const void* W1, const void* W2) {
    int rc = check_args(s, o, b);
    if (rc) return rc;
    if (!o->logits_given && (rc = gate_logits_check(s, x, Wg, b->logits, o->jitter_eps))) return rc;
    if ((rc = route_check(s, o->groups, b->logits, b->probs, b->expert_idx, b->gate_w, b->slot, b->expert_count,
                          b->expert_demand, b->slot_src, b->ws, b->ws_bytes))) return rc;
    if (o->forward_only && !b->utilisation) return MOE_ERR_NULL;
    if (o->aux_coef != 0.0f &&
        (rc = aux_loss_check(s, b->probs, b->expert_idx, b->first_frac, b->mean_prob, b->aux_loss, b->ws, b->ws_bytes))) return rc;
    if ((rc = dispatch_tokens_check(s, x, b->expert_idx, b->slot, b->xd))) return rc;
    if ((rc = ffn_fwd_check(s, b->xd, b->expert_count, W1, W2, o->drop_p > 0.0f ? o->drop_p : 0.0f, b->h, b->dact, b->yd))) return rc;
    return combine_fwd_check(s, b->yd, b->expert_idx, b->slot, b->y);
}

static int check_bwd(const moe_shape* s, const moe_layer_options* o, const moe_layer_buffers* b, const void* x,
                     const float* Wg, const void* W1, const void* W2, const void* dy) {
    int rc = check_args(s, o, b);
    if (rc) return rc;
    if ((rc = combine_gate_bwd_check(s, dy, b->yd, b->expert_idx, b->slot, b->gate_w, b->probs, b->dyd, b->dgate_w, b->dlogits))) return rc;
    if ((rc = ffn_bwd_check(s, b->dyd, b->xd, b->h, b->dact, b->expert_count, W1, W2, b->dxd, b->dW1, b->dW2, b->ws, b->ws_bytes))) return rc;
    // without first_frac moe_combine_gate_bwd would leave the balancing loss's gradient out
    if (!b->dx || (o->aux_coef != 0.0f && !b->first_frac)) return MOE_ERR_NULL;
    return gate_logits_bwd_check(s, x, Wg, b->dlogits, o->jitter_eps, b->dWg, b->ws, b->ws_bytes);
}

extern "C" int moe_layer_fwd(const moe_shape* s, const moe_layer_options* o, const moe_layer_buffers* b,
                             const void* x, const float* Wg, const float* bias_or_null, const void* W1,
                             const void* W2, const float* rts_keys_or_null, void* stream) {
    int rc = check_fwd(s, o, b, x, Wg, W1, W2);
    if (!rc && !o->logits_given)
        rc = moe_gate_logits_jitter(s, x, Wg, bias_or_null, o->jitter_eps, o->seed, b->logits, stream);
    if (rc) return rc;
    if (o->forward_only)
        rc = moe_gate_route_counted(s, o->groups, b->logits, rts_keys_or_null, b->probs, b->expert_idx, b->gate_w, b->slot,
                                    b->expert_count, b->expert_demand, b->slot_src, b->utilisation, b->ws, b->ws_bytes, stream);
    else
        rc = moe_gate_route_grouped(s, o->groups, b->logits, rts_keys_or_null, b->probs, b->expert_idx, b->gate_w, b->slot,
                                    b->expert_count, b->expert_demand, b->slot_src, b->ws, b->ws_bytes, stream);
    if (!rc && o->aux_coef != 0.0f)
        rc = moe_aux_loss(s, b->probs, b->expert_idx, b->first_frac, b->mean_prob, b->aux_loss, b->ws, b->ws_bytes, stream);
    if (!rc) rc = moe_dispatch_tokens(s, x, b->expert_idx, b->slot, b->xd, stream);    // reads every token row once
    if (rc) return rc;
    if (o->drop_p > 0.0f)
        rc = moe_expert_ffn_fwd_dropout(s, b->xd, b->expert_count, W1, W2, o->drop_p, o->seed, b->h, b->dact, b->yd, stream);
    else
        rc = moe_expert_ffn_fwd(s, b->xd, b->expert_count, W1, W2, b->h, b->dact, b->yd, stream);
    if (!rc) rc = moe_combine_fwd(s, b->yd, b->expert_idx, b->slot, b->gate_w, b->y, stream);
    return rc;
}

extern "C" int moe_layer_bwd(const moe_shape* s, const moe_layer_options* o, const moe_layer_buffers* b,
                             const void* x, const float* Wg, const void* W1, const void* W2, const void* dy,
                             void* stream) {
    int rc = check_bwd(s, o, b, x, Wg, W1, W2, dy);
    if (!rc)
        rc = moe_combine_gate_bwd(s, dy, b->yd, b->expert_idx, b->slot, b->gate_w, b->probs,
                                  o->aux_coef != 0.0f ? b->first_frac : nullptr, o->aux_coef, b->dyd, b->dgate_w, b->dlogits, stream);
    if (!rc)
        rc = moe_expert_ffn_bwd(s, b->dyd, b->xd, b->h, b->dact, b->expert_count, W1, W2, b->dxd, b->dW1, b->dW2, b->ws,
                                b->ws_bytes, stream);
    // dispatch's backward (combine with unit weights) and the gate projection's backward in one call
    if (!rc)
        rc = moe_dispatch_gate_logits_bwd(s, x, Wg, b->dlogits, b->dxd, b->expert_idx, b->slot, o->jitter_eps, o->seed,
                                          b->dWg, b->dx, b->ws, b->ws_bytes, stream);
    return rc;
}
