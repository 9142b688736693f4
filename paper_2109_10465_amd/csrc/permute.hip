// Dispatch into per-expert capacity buffers and the gate-weighted combine
// (Sec. 3.1: fixed-shape per-expert buffers; dropped tokens get a zero output
// row).  Pure HBM traffic: every row moves as 16-byte vectors, one wavefront
// per row, fp32 math, no atomics (each output row has exactly one writer).
#include "moe_common.h"

#ifndef ROWS_PER_WG
#define ROWS_PER_WG 4  // one wave per row, 4 waves per workgroup
#endif

// xd[e,s,:] = x[slot_src[e,s]/k, :]   for s < expert_count[e]
template <typename T>
__global__ __launch_bounds__(64 * ROWS_PER_WG) void dispatch_kernel(int d, int k, int C, int n_rows, int n_cand,
                                                       const T* __restrict__ x,
                                                       const int32_t* __restrict__ slot_src,
                                                       const int32_t* __restrict__ expert_count,
                                                       T* __restrict__ xd) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * ROWS_PER_WG + (threadIdx.x >> 6);
    if (row >= n_rows) return;
    const int e = row / C, s = row - e * C;
    if (s >= expert_count[e]) return;
    // a slot in use always names a candidate; the check only matters when the routing was
    // fed non-finite keys (two candidates can then share a rank and leave a slot unwritten)
    const int cand = slot_src[row];
    if ((unsigned)cand >= (unsigned)n_cand) return;
    const int t = cand / k;
    const uint4* src = reinterpret_cast<const uint4*>(x + (size_t)t * d);
    uint4* dst = reinterpret_cast<uint4*>(xd + (size_t)row * d);
    const int nvec = d * (int)sizeof(T) / 16;
    for (int v = lane; v < nvec; v += 64) dst[v] = src[v];
}

// The same copy, token-major: one wave per token reads x[t,:] once and writes it to the
// slot of each kept choice (the slot-major kernel above reads a token's row once per
// kept choice).  xd[expert_idx[t,j], slot[t,j], :] = x[t,:] for slot[t,j] >= 0.
template <typename T>
__global__ __launch_bounds__(64 * ROWS_PER_WG) void dispatch_tokens_kernel(int Tn, int d, int k, int E, int C,
                                                                           const T* __restrict__ x,
                                                                           const int32_t* __restrict__ expert_idx,
                                                                           const int32_t* __restrict__ slot,
                                                                           T* __restrict__ xd) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROWS_PER_WG + (threadIdx.x >> 6);
    if (t >= Tn) return;
    uint4* dst[2] = {nullptr, nullptr};
    for (int j = 0; j < k; ++j) {
        const int s = slot[(size_t)t * k + j];
        const int e = expert_idx[(size_t)t * k + j];
        // ids and slots come from the routing call; anything else is skipped, never dereferenced
        if (s >= 0 && s < C && (unsigned)e < (unsigned)E) dst[j] = reinterpret_cast<uint4*>(xd + ((size_t)e * C + s) * d);
    }
    if (!dst[0] && !dst[1]) return;      // fully dropped token: nothing to copy, x[t] is not read
    const uint4* src = reinterpret_cast<const uint4*>(x + (size_t)t * d);
    const int nvec = d * (int)sizeof(T) / 16;
    for (int v = lane; v < nvec; v += 64) {
        const uint4 q = src[v];
        if (dst[0]) dst[0][v] = q;
        if (dst[1]) dst[1][v] = q;
    }
}

// y[t,:] = sum_j [slot>=0] g_j * yd[e_j, slot_j, :]
template <typename T>
__global__ __launch_bounds__(64 * ROWS_PER_WG) void combine_fwd_kernel(int Tn, int d, int k, int C,
                                                          const T* __restrict__ yd,
                                                          const int32_t* __restrict__ expert_idx,
                                                          const int32_t* __restrict__ slot,
                                                          const float* __restrict__ gate_w,
                                                          T* __restrict__ y) {
    constexpr int CN = Chunk<T>::N;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROWS_PER_WG + (threadIdx.x >> 6);
    if (t >= Tn) return;
    const T* src[2] = {nullptr, nullptr};
    float g[2] = {0.0f, 0.0f};
    for (int j = 0; j < k; ++j) {
        const int s = slot[(size_t)t * k + j];
        if (s >= 0) {
            src[j] = yd + ((size_t)expert_idx[(size_t)t * k + j] * C + s) * d;
            g[j] = gate_w ? gate_w[(size_t)t * k + j] : 1.0f;
        }
    }
    const int nvec = d / CN;
    for (int v = lane; v < nvec; v += 64) {
        float acc[CN];
#pragma unroll
        for (int i = 0; i < CN; ++i) acc[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (src[j]) {
                float a[CN];
                Chunk<T>::load(src[j] + (size_t)v * CN, a);
#pragma unroll
                for (int i = 0; i < CN; ++i) acc[i] = fmaf(g[j], a[i], acc[i]);
            }
        }
        Chunk<T>::store(y + (size_t)t * d + (size_t)v * CN, acc);
    }
}

// dyd[e,s,:] = g_j * dy[t,:];  dgate_w[t,j] = <dy[t,:], yd[e,s,:]>
// GATE: the token's dlogits row follows at once (the derivative of the gate weights and the softmax,
// with aux_c * first_frac[e] added to dp[t,e] when first_frac is given): the wave has the token's
// dgate_w, so the row costs one read of probs and one write instead of a launch of its own
// (T = 32768, E = 128: 17.8 + 11.9 us apart, 25.8 together; T = 256, E = 4: 3.2 + 4.6 apart, 3.8 together).
template <typename T, bool GATE>
__global__ __launch_bounds__(64 * ROWS_PER_WG) void combine_bwd_kernel(int Tn, int d, int E, int k, int C,
                                                          const T* __restrict__ dy,
                                                          const T* __restrict__ yd,
                                                          const int32_t* __restrict__ expert_idx,
                                                          const int32_t* __restrict__ slot,
                                                          const float* __restrict__ gate_w,
                                                          const float* __restrict__ probs,
                                                          const float* __restrict__ first_frac, float aux_c,
                                                          T* __restrict__ dyd, float* __restrict__ dgate_w,
                                                          float* __restrict__ dlogits) {
    constexpr int CN = Chunk<T>::N;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROWS_PER_WG + (threadIdx.x >> 6);
    if (t >= Tn) return;
    size_t off[2] = {0, 0};
    int ev[2] = {-1, -1};
    bool kept[2] = {false, false};
    float g[2] = {0.0f, 0.0f}, dot[2] = {0.0f, 0.0f};
    for (int j = 0; j < k; ++j) {
        const int s = slot[(size_t)t * k + j];
        ev[j] = expert_idx[(size_t)t * k + j];
        if (s >= 0) {
            kept[j] = true;
            off[j] = ((size_t)ev[j] * C + s) * d;
            g[j] = gate_w[(size_t)t * k + j];
        }
    }
    // the token's probabilities are requested before the rows: four consecutive experts per lane
    const int e4 = 4 * lane;
    const bool vec = (E & 3) == 0;
    float pe[4] = {0.f, 0.f, 0.f, 0.f}, ff[4] = {0.f, 0.f, 0.f, 0.f}, pc[2] = {0.f, 0.f};
    if constexpr (GATE) {
        const float* pr = probs + (size_t)t * E;
        if (vec) {
            if (e4 < E) {
                const float4 q = *reinterpret_cast<const float4*>(pr + e4);
                pe[0] = q.x; pe[1] = q.y; pe[2] = q.z; pe[3] = q.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) pe[i] = e4 + i < E ? pr[e4 + i] : 0.0f;
        }
        if (first_frac) {
#pragma unroll
            for (int i = 0; i < 4; ++i) ff[i] = e4 + i < E ? aux_c * first_frac[e4 + i] : 0.0f;
        }
        for (int j = 0; j < k; ++j) pc[j] = pr[ev[j]];
    }
    if (kept[0] || kept[1]) {
        const int nvec = d / CN;
        for (int v = lane; v < nvec; v += 64) {
            float a[CN];
            Chunk<T>::load(dy + (size_t)t * d + (size_t)v * CN, a);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (kept[j]) {
                    float b[CN], o[CN];
                    Chunk<T>::load(yd + off[j] + (size_t)v * CN, b);
#pragma unroll
                    for (int i = 0; i < CN; ++i) {
                        dot[j] = fmaf(a[i], b[i], dot[j]);
                        o[i] = g[j] * a[i];
                    }
                    Chunk<T>::store(dyd + off[j] + (size_t)v * CN, o);
                }
            }
        }
    }
    float dg[2] = {0.0f, 0.0f};
    for (int j = 0; j < k; ++j) {
        const float tot = wave_sum(dot[j]);
        dg[j] = kept[j] ? tot : 0.0f;
        if (lane == 0) dgate_w[(size_t)t * k + j] = dg[j];
    }
    if constexpr (GATE) {
        float dp0 = dg[0], dp1 = 0.0f;
        if (k == 2) {
            const float S = pc[0] + pc[1];
            dp0 = pc[1] * (dg[0] - dg[1]) / (S * S);
            dp1 = pc[0] * (dg[1] - dg[0]) / (S * S);
        }
        float sum = pc[0] * dp0 + pc[1] * dp1;       // sum over experts of p dp
        if (first_frac) {
            float part = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) part = fmaf(pe[i], ff[i], part);
            sum += wave_sum(part);
        }
        float out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float dp = ff[i];
            if (e4 + i == ev[0]) dp += dp0;
            if (e4 + i == ev[1]) dp += dp1;
            out[i] = pe[i] * (dp - sum);
        }
        float* dl = dlogits + (size_t)t * E;
        if (vec) {
            if (e4 < E) *reinterpret_cast<float4*>(dl + e4) = make_float4(out[0], out[1], out[2], out[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (e4 + i < E) dl[e4 + i] = out[i];
        }
    }
}

extern "C" int moe_dispatch(const moe_shape* shape, const void* x, const int32_t* slot_src,
                            const int32_t* expert_count, void* xd, void* stream) {
    int rc = check_shape(shape);
    if (rc) return rc;
    if (!x || !slot_src || !expert_count || !xd) return MOE_ERR_NULL;
    const int n_rows = shape->E * shape->capacity;
    const int grid = ceil_div(n_rows, ROWS_PER_WG);
    hipStream_t st = (hipStream_t)stream;
    if (shape->dtype == MOE_BF16)
        dispatch_kernel<bf16_t><<<grid, 64 * ROWS_PER_WG, 0, st>>>(shape->d_model, shape->k, shape->capacity, n_rows, shape->T * shape->k,
                                                      (const bf16_t*)x, slot_src, expert_count, (bf16_t*)xd);
    else
        dispatch_kernel<float><<<grid, 64 * ROWS_PER_WG, 0, st>>>(shape->d_model, shape->k, shape->capacity, n_rows, shape->T * shape->k,
                                                     (const float*)x, slot_src, expert_count, (float*)xd);
    return launch_status();
}

int dispatch_tokens_check(const moe_shape* s, const void* x, const int32_t* expert_idx, const int32_t* slot, const void* xd) {
    const int rc = shape_status(s);
    return rc ? rc : x && expert_idx && slot && xd ? MOE_OK : MOE_ERR_NULL;
}

extern "C" int moe_dispatch_tokens(const moe_shape* shape, const void* x, const int32_t* expert_idx,
                                   const int32_t* slot, void* xd, void* stream) {
    const int rc = begin_call(dispatch_tokens_check(shape, x, expert_idx, slot, xd));
    if (rc) return rc;
    const int grid = ceil_div(shape->T, ROWS_PER_WG);
    hipStream_t st = (hipStream_t)stream;
    if (shape->dtype == MOE_BF16)
        dispatch_tokens_kernel<bf16_t><<<grid, 64 * ROWS_PER_WG, 0, st>>>(shape->T, shape->d_model, shape->k, shape->E, shape->capacity,
                                                                 (const bf16_t*)x, expert_idx, slot, (bf16_t*)xd);
    else
        dispatch_tokens_kernel<float><<<grid, 64 * ROWS_PER_WG, 0, st>>>(shape->T, shape->d_model, shape->k, shape->E, shape->capacity,
                                                                (const float*)x, expert_idx, slot, (float*)xd);
    return launch_status();
}

int combine_fwd_check(const moe_shape* s, const void* yd, const int32_t* expert_idx, const int32_t* slot, const void* y) {
    const int rc = shape_status(s);
    return rc ? rc : yd && expert_idx && slot && y ? MOE_OK : MOE_ERR_NULL;
}

extern "C" int moe_combine_fwd(const moe_shape* shape, const void* yd, const int32_t* expert_idx,
                               const int32_t* slot, const float* gate_w_or_null, void* y,
                               void* stream) {
    const int rc = begin_call(combine_fwd_check(shape, yd, expert_idx, slot, y));
    if (rc) return rc;
    const int grid = ceil_div(shape->T, ROWS_PER_WG);
    hipStream_t st = (hipStream_t)stream;
    if (shape->dtype == MOE_BF16)
        combine_fwd_kernel<bf16_t><<<grid, 64 * ROWS_PER_WG, 0, st>>>(shape->T, shape->d_model, shape->k, shape->capacity,
                                                         (const bf16_t*)yd, expert_idx, slot, gate_w_or_null, (bf16_t*)y);
    else
        combine_fwd_kernel<float><<<grid, 64 * ROWS_PER_WG, 0, st>>>(shape->T, shape->d_model, shape->k, shape->capacity,
                                                        (const float*)yd, expert_idx, slot, gate_w_or_null, (float*)y);
    return launch_status();
}

template <bool GATE>
static void launch_combine_bwd(const moe_shape* s, const void* dy, const void* yd, const int32_t* expert_idx,
                               const int32_t* slot, const float* gate_w, const float* probs, const float* first_frac,
                               float aux_coef, void* dyd, float* dgate_w, float* dlogits, void* stream) {
    const int grid = ceil_div(s->T, ROWS_PER_WG);
    const float c = aux_coef * (float)s->E / (float)s->T;
    hipStream_t st = (hipStream_t)stream;
    if (s->dtype == MOE_BF16)
        combine_bwd_kernel<bf16_t, GATE><<<grid, 64 * ROWS_PER_WG, 0, st>>>(s->T, s->d_model, s->E, s->k, s->capacity,
            (const bf16_t*)dy, (const bf16_t*)yd, expert_idx, slot, gate_w, probs, first_frac, c, (bf16_t*)dyd, dgate_w, dlogits);
    else
        combine_bwd_kernel<float, GATE><<<grid, 64 * ROWS_PER_WG, 0, st>>>(s->T, s->d_model, s->E, s->k, s->capacity,
            (const float*)dy, (const float*)yd, expert_idx, slot, gate_w, probs, first_frac, c, (float*)dyd, dgate_w, dlogits);
}

extern "C" int moe_combine_bwd(const moe_shape* shape, const void* dy, const void* yd,
                               const int32_t* expert_idx, const int32_t* slot, const float* gate_w,
                               void* dyd, float* dgate_w, void* stream) {
    int rc = check_shape(shape);
    if (rc) return rc;
    if (!dy || !yd || !expert_idx || !slot || !gate_w || !dyd || !dgate_w) return MOE_ERR_NULL;
    launch_combine_bwd<false>(shape, dy, yd, expert_idx, slot, gate_w, nullptr, nullptr, 0.0f, dyd, dgate_w, nullptr, stream);
    return launch_status();
}

// One pass for combine and gate backward, or two?  One saves a launch (5 us) and a read of dgate_w, but it has a wave
// per token for a dlogits row that a few lanes write, which shows once there are many tokens of short rows.
// Measured, one pass against two, us:
//   bf16, E = 32, top-2: T = 16384, d = 64 11.2 and 11.6, T = 24576, d = 128 16.5 and 15.8, T = 32768, d = 64 20.2 and 18.2, d = 512
//     30.9 and 31.2; T = 65536, d = 512 81.4 and 74.4; T = 131072, d = 256 132.6 and 115.3, fp32, d = 512 (2 KB rows): the same
//   bf16, E = 16, top-1: T = 32768, d = 64 14.0 and 14.0; T = 65536, d = 128 28.2 and 25.7; E = 64: 4 % faster in one pass
//   E = 256: one pass is the faster one throughout (T = 131072, d = 128, top-2: 6 %)
static bool two_passes_win(const moe_shape* s) {
    const int64_t choices = (int64_t)s->T * s->k;
    const size_t row = s->d_model * elem_bytes(s->dtype);
    return s->E <= 32 * s->k && (choices >= 131072 ? row <= 1024 : choices >= 49152 && row <= 512);
}

// measurement aid: passes of moe_combine_gate_bwd over the tokens
extern "C" int moe_combine_gate_bwd_launches(const moe_shape* shape) {
    const int rc = shape_status(shape);
    return rc ? rc : two_passes_win(shape) ? 2 : 1;
}

int combine_gate_bwd_check(const moe_shape* s, const void* dy, const void* yd, const int32_t* expert_idx,
                           const int32_t* slot, const float* gate_w, const float* probs, const void* dyd,
                           const float* dgate_w, const float* dlogits) {
    const int rc = shape_status(s);
    if (rc) return rc;
    return dy && yd && expert_idx && slot && gate_w && probs && dyd && dgate_w && dlogits ? MOE_OK : MOE_ERR_NULL;
}

extern "C" int moe_combine_gate_bwd(const moe_shape* shape, const void* dy, const void* yd,
                                    const int32_t* expert_idx, const int32_t* slot, const float* gate_w,
                                    const float* probs, const float* first_frac_or_null, float aux_coef,
                                    void* dyd, float* dgate_w, float* dlogits, void* stream) {
    const int rc = begin_call(combine_gate_bwd_check(shape, dy, yd, expert_idx, slot, gate_w, probs, dyd, dgate_w, dlogits));
    if (rc) return rc;
    // (in one pass every wave has its token's probabilities before it writes the row: dlogits may be probs itself)
    if (two_passes_win(shape) && dlogits != probs) {
        launch_combine_bwd<false>(shape, dy, yd, expert_idx, slot, gate_w, nullptr, nullptr, 0.0f, dyd, dgate_w, nullptr, stream);
        return first_frac_or_null
            ? moe_gate_bwd_aux(shape, dgate_w, probs, expert_idx, slot, first_frac_or_null, aux_coef, dlogits, stream)
            : moe_gate_bwd(shape, dgate_w, probs, expert_idx, slot, dlogits, stream);
    }
    launch_combine_bwd<true>(shape, dy, yd, expert_idx, slot, gate_w, probs, first_frac_or_null, aux_coef, dyd, dgate_w,
                             dlogits, stream);
    return launch_status();
}
