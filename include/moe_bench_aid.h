/*
 * moe_bench_aid.h - measurement aid shipped with the MoE layer library; NOT part of
 * the layer's ABI (that is moe_hip.h): what the chip sustains on the matrix pipe, which
 * bench.py prints beside the published peak, and which kernel a dispatch rule chooses for
 * a shape, for the tests of the rules and for whoever times the calls.
 */
#ifndef MOE_BENCH_AID_H
#define MOE_BENCH_AID_H

#include "moe_hip.h"

#ifdef __cplusplus
extern "C" {
#endif

/* n_workgroups x 4 waves each issue iters x 8 independent v_mfma_f32_32x32x16_bf16 on register-resident operands
 * (random_operands != 0: seeded pseudo-random values, else all-equal ones).
 * Work = n_workgroups * 4 * iters * 8 * 32768 flop; the caller times it.
 * out: n_workgroups * 256 floats, written once so that the loop is not dead code. */
int moe_microbench_mfma_bf16(int32_t n_workgroups, int32_t iters, int32_t random_operands, float* out,
                             void* stream);

/* Launches of one routing call (moe_gate_route, _grouped, _counted): 1 = one workgroup does it
 * all, 3 = gate, placement and ranking.  Host function; a moe_status on an invalid shape. */
int moe_route_launches(const moe_shape* shape, int32_t n_groups, int32_t has_keys);

/* 32-token tiles that share a workgroup of the gate projection (moe_gate_logits) of at most 32
 * experts: 1 or 2 (1 for fp32).  Host function. */
int moe_gate_logits_token_tiles(const moe_shape* shape);

/* Launches of the projection's backward (moe_gate_logits_bwd and the calls built on it): 1 = dWg and
 * dx together, else dWg in two and dx in one.  Host function. */
int moe_gate_logits_bwd_launches(const moe_shape* shape, int32_t with_dx, float jitter_eps);

/* Token chunks, each with a partial sum of dWg of its own, of the form with several launches. */
int moe_gate_logits_bwd_chunks(const moe_shape* shape, float jitter_eps);

/* Launches of moe_combine_gate_bwd: 1 = one pass over the tokens, 2 = combine, then gate. */
int moe_combine_gate_bwd_launches(const moe_shape* shape);

/* Tile side (32, 64, 128 or 256) and groups of four waves that share a tile (1 or 2), for each of the
 * expert FFN's four launches: xd W1, h W2, dz with dW2, dxd with dW1. */
int moe_expert_ffn_tiles(const moe_shape* shape, int32_t* side, int32_t* wave_groups);

/* For the same four launches: 1 where the tile is fp32's 32 x 32 one, whose reduction a workgroup's four waves share,
 * 0 elsewhere. */
int moe_expert_ffn_parts(const moe_shape* shape, int32_t* parts);

/* For the same four launches: 1 where every workgroup takes one tile whose place does not depend on the experts' row
 * counts, 0 where workgroups walk the tiles that the counts leave; and how many workgroups there are. */
int moe_expert_ffn_direct(const moe_shape* shape, int32_t* direct, int32_t* workgroups);

#ifdef __cplusplus
}
#endif
#endif /* MOE_BENCH_AID_H */
