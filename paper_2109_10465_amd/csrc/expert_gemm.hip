// Grouped expert GEMMs on the MFMA matrix cores: the per-expert feed-forward
// block d_model -> d_ff -> d_model, forward and backward (Sec. 4.2 "Model
// details"; Sec. 2.3: these matmuls are where the layer's time goes).
//
// One kernel template serves the six contractions.  Per expert e with
// n_e = expert_count[e] rows in use:
//   forward   z = xd W1        (rows x d)(d x f)     epilogue: h = act(z), a = act'(z)
//             yd = h W2        (rows x f)(f x d)
//   backward  dz = (dyd W2^T) .* a
//             dxd = dz W1^T
//             dW2 = h^T dyd    (f x rows)(rows x d)  fp32 output, K = rows
//             dW1 = xd^T dz    (d x rows)(rows x f)
// Each operand is described as a (row index r, reduction index k) array that is
// either k-contiguous in memory (KC) or r-contiguous (!KC); no transposed copy
// of any tensor is ever materialised.
//
// Three kernels: a large-tile one for bf16 (below), one with smaller tiles for everything
// else and one for fp32's smallest products (their own comments say what for); launch_gemm
// chooses by the number of tiles.
//
// Structure of a large-tile workgroup (8 waves, 2 x 4, two per SIMD; one persistent
// workgroup per CU):
//   * walks BM x BN output tiles.  Only tiles that hold rows exist; the expert-major
//     tile sequence is dealt block-cyclically, a block of as many consecutive tiles
//     as an XCD has workgroups going to one XCD (workgroup w runs on XCD w % 8), so
//     the tiles an XCD works on at one time are neighbours and share operand panels
//     in its L2, every workgroup gets the same number of a product's tiles up to one
//     (a launch's second product: fewer where the first one's tiles are long), and a
//     heavily loaded expert is spread over all XCDs.  The slabs of all tiles of a
//     workgroup form one stream through the LDS ring: the next tile's first slabs
//     arrive under the current tile's epilogue;
//   * streams BK-deep slabs of both operands with 16-byte buffer loads that write
//     straight into LDS (no register staging).  bf16: BK = 64 (a k-contiguous operand
//     is fetched in 128-byte row pieces), two 64 KB stages.  The B half of a stage is
//     released early: a wave holds few B fragments, so it reads those of all four
//     k-steps during the slab's first step and the half is refilled three k-steps
//     before the A half - requests are in flight nearly all the time instead of in
//     one burst per slab, and B has 1.75 slab periods to arrive.  The slab's offset
//     is applied to the buffer descriptor (scalar work); the descriptor's range check
//     supplies the zero fill for rows >= n_e, so the loop has no branches.  LDS tiles
//     are unpadded and XOR-swizzled in 16-byte units (fragment reads are free of bank
//     conflicts);
//   * each wave accumulates (BM/2) x (BN/NWN) in 32x32 MFMA tiles; !KC
//     operands are read from LDS with the transposing ds_read_b64_tr_b16.  A wave
//     issues strictly in order and an MFMA holds it for the MFMA's 32 cycles, so the
//     matrix pipe is kept busy by the SIMD's other wave; loads and fragment reads are
//     dealt evenly over the MFMA slots for that reason;
//   * the epilogue passes the accumulators through LDS so that every global
//     store is a full 8/16-byte vector along the row; the activation and its
//     derivative are evaluated once, in the forward epilogue (code kept in a
//     rolled loop), and the backward epilogue only multiplies by the saved
//     derivative, which it fetched into registers before the main loop;
//   * the backward's four products run as two launches of two independent products
//     each (dz with dW2, dxd with dW1): one walk over the tiles of the first, then of
//     the second (6 experts of 1440 rows, d = 776, f = 3080: 174 -> 143 us for the second
//     pair against two walks that both start at the first workgroup).
#include <math.h>
#include <type_traits>
#include "moe_common.h"

// the large bf16 tile: rows, columns, slab depth, wavefronts along N
enum { BIG_M = 256, BIG_N = 256, BIG_K = 64, BIG_WN = 4 };

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

enum { EPI_STORE = 0, EPI_H_DACT = 1, EPI_MUL = 2, EPI_F32 = 3, EPI_H = 4 };   // EPI_H: activation only (forward-only use)

struct GemmArgs {
    const void* A; const void* B;
    void* out0; void* out1; const void* aux;
    const int32_t* expert_count;
    long long strideA, strideB, strideO;  // elements per expert
    int lda, ldb, ldo;
    int M, N, K;      // extents; the one bounded by expert_count is an upper limit
    int var_k;        // 0: rows (M) bounded by expert_count; 1: K bounded by it
    int tiles_m, tiles_n, E;
    // smaller tiles, where each that there could be has a workgroup of its own (set_direct): this product's are an XCD's
    // workgroups from direct_first on, direct_count tiles in all (0: by the experts' row counts); t / d is the upper half of t * inv
    int direct_first, direct_count;
    uint32_t inv_expert, inv_m;
    int lead;         // second product of a launch: what a tile of the first one lasts, in reduction entries (TileWalk::follow)
    // expert dropout in the activation epilogue (drop_thr = 0: off): an element is dropped when its
    // noise word < drop_thr, kept ones are scaled by drop_scale = 1 / (1 - p)
    uint32_t drop_thr;
    float drop_scale;
    uint64_t seed;
};

template <typename T> struct Mma;
template <> struct Mma<bf16_t> {
    static constexpr int FE = 8;      // elements per lane per operand
    static constexpr int KSTEP = 16;  // reduction depth of one MFMA
    typedef bf16x8_t frag;
    __device__ static __forceinline__ f32x16_t mma(frag a, frag b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};
#define OOB_OFFSET 0x80000000u  // beyond any descriptor this kernel builds (slices < 2 GiB)

// LDS tile of one operand: BR rows (r) x BK reduction entries, unpadded, as
// 16-byte slots; slot p is filled by thread p % NT in its (p / NT)-th load.
//   KC : LDS row = r (BK entries),  slot = r*CPR + (chunk ^ swz(r))
//   !KC: LDS row = k (BR entries),  slot = k*CPR + (chunk ^ swz(k))
// swz: KC  -> consecutive rows that share a 256-byte bank window get distinct
//             chunk positions (16-byte fragment reads of 16 rows hit 64 banks);
//      !KC -> rows k, k+1, k+2, k+3 are shifted by 64 bytes each (the
//             transposing 8-byte reads of 4 rows x 64 bytes hit 64 banks).
template <typename T, int BR, int BK, bool KC, int NT> struct Tile {
    static constexpr int CN = 16 / (int)sizeof(T);           // elements per slot
    static constexpr int CPR = (KC ? BK : BR) / CN;          // slots per LDS row
    static constexpr int ROWS = KC ? BR : BK;
    static constexpr int SLOTS = ROWS * CPR;
    static constexpr int PER_THREAD = SLOTS / NT;
    static constexpr int BYTES = SLOTS * 16;
    static constexpr int WIN = CPR >= 16 ? 1 : 16 / CPR;     // rows per 256-byte window
    static constexpr bool IS_KC = KC;
    static_assert(SLOTS % NT == 0, "tile must be a multiple of the workgroup size in slots");
    static_assert((CPR & (CPR - 1)) == 0, "slots per row must be a power of two");

    __device__ static __forceinline__ int swz(int row) {
        if (KC) return (row / WIN) & (CPR - 1);
        return CPR >= 16 ? ((row & 3) << 2) : ((row >> 1 & 1) << 2) & (CPR - 1);
    }

    // Per-thread load plan: byte offset of each of its slots at reduction offset 0
    // (OOB_OFFSET where the non-linear guard already fails) and, for KC, the
    // reduction column of the slot (its guard depends on the slab).
    struct Plan { uint32_t voff[PER_THREAD]; int kcol[PER_THREAD]; };
    __device__ static __forceinline__ void plan(Plan& pl, int ld, int r0, int r_lim) {
#pragma unroll
        for (int i = 0; i < PER_THREAD; ++i) {
            const int p = threadIdx.x + i * NT;
            const int row = p / CPR, c = (p % CPR) ^ swz(row);
            if (KC) {
                pl.voff[i] = (uint32_t)((r0 + row) * ld + c * CN) * (uint32_t)sizeof(T);
                pl.kcol[i] = c * CN;
            } else {
                const int r = r0 + c * CN;
                pl.voff[i] = r < r_lim ? (uint32_t)(row * ld + r) * (uint32_t)sizeof(T) : OOB_OFFSET;
                pl.kcol[i] = 0;
            }
        }
    }
    // Descriptor range = the linear guard: KC rows < r_lim, !KC reduction rows < k_lim.
    __device__ static __forceinline__ u32x4_t desc(const T* g, int ld, int r_lim, int k_lim) {
        return make_desc(g, (uint32_t)(KC ? r_lim : k_lim) * (uint32_t)ld * (uint32_t)sizeof(T));
    }
    // Byte shift of the slab at reduction offset k0 inside the operand; it is applied to the
    // descriptor (scalar work, once per slab), not to every lane's offset.
    __device__ static __forceinline__ uint32_t slab_shift(int ld, int k0) {
        return (uint32_t)(KC ? k0 : k0 * ld) * (uint32_t)sizeof(T);
    }
    // The descriptor of one slab: base moved to the slab's first reduction entry.  For an
    // r-contiguous operand the range shrinks by the same amount, so that "reduction row < k_lim"
    // stays the descriptor's range check; for a k-contiguous operand the range (rows < r_lim)
    // is kept - every in-range row stays inside the tensor as long as the slab does.
    __device__ static __forceinline__ u32x4_t slab_desc(u32x4_t d, uint32_t shift) {
        const uint64_t base = ((uint64_t)(d[1] & 0xffffu) << 32 | d[0]) + shift;
        d[0] = (uint32_t)base;
        d[1] = (d[1] & 0xffff0000u) | (uint32_t)(base >> 32);
        if (!KC) d[2] = d[2] > shift ? d[2] - shift : 0u;
        return d;
    }
    // The i-th of this thread's loads of the slab whose descriptor is ds, into the stage at lds_base.
    // KG: the reduction length is not a multiple of BK, so a k-contiguous operand needs a per-lane
    // guard in its last slab (an r-contiguous one never does: the descriptor's range is that guard).
    template <bool KG>
    __device__ static __forceinline__ void issue_one(const Plan& pl, u32x4_t ds, int k0, int k_lim, uint32_t lds_base, int i) {
        const uint32_t wave_base = lds_base + (threadIdx.x >> 6) * 1024;
        uint32_t off = pl.voff[i];
        if (KC && KG) off = pl.kcol[i] + k0 < k_lim ? off : OOB_OFFSET;
        load_to_lds(ds, off, __builtin_amdgcn_readfirstlane(wave_base + i * NT * 16));
    }
    // LDS -> MFMA operand for the 32 tile rows rbase..rbase+31 (this lane: row
    // rbase + lane%32), reduction step ks; lane group g = lane/32 holds the
    // reduction entries ks*KSTEP + FE*g .. + FE-1.
    __device__ static __forceinline__ typename Mma<T>::frag frag(const unsigned char* s, int rbase, int ks, int lane) {
        constexpr int FE = Mma<T>::FE;
        const int g = lane >> 5, l32 = lane & 31;
        const int k = ks * Mma<T>::KSTEP + FE * g;
        if constexpr (sizeof(T) == 2) {
            if constexpr (KC) {
                const int row = rbase + l32;
                const int slot = row * CPR + ((k / CN) ^ swz(row));
                return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(s + slot * 16));
            } else {
                // ds_read_b64_tr_b16: within 16 lanes, lane s supplies the address of 4
                // consecutive r at reduction row (s/4); lane l receives, for its own
                // r = 4*(l/4)+(l%4) of those 16, the entries of 4 consecutive rows.
                const int sl = lane & 15;
                const int kr = k + (sl >> 2);
                const int col = rbase + (l32 & 16) + 4 * (sl & 3);
                const int slot = kr * CPR + ((col / CN) ^ swz(kr));
                const unsigned char* p = s + slot * 16 + (col % CN) * 2;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p);
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p + 4 * CPR * 16));
                const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(bf16x8_t, v);
            }
        }
    }
};

// ---- activation in the forward epilogue ---------------------------------------
// h = act(z) and a = act'(z) together.
// fp32 tensors: the normal cdf Phi from two fits that meet at |z| = 1.0625, without erff and expf (about 32
// instructions against about 100; forward pair at 8 experts of 1024 rows, d = 512, f = 2048: 201.3 us against
// 204.7).  Inside, Phi(z) = 1/2 + z C(z^2), one rounding at the size of the result; outside, Phi(-t) = phi(t) M(t)
// with Mills' ratio M as a (3,4) rational function, small against the 1 or 0 that it is taken from.  The
// density's exponent keeps what its own rounding leaves.
//   C: least squares in z^2 on Chebyshev nodes of [0, 1.129], weight |z| + 0.05, each coefficient rounded to fp32
//      before the next ones are fitted (error of z C: 1.5e-9).
//   M: linearised least squares on Chebyshev nodes of [1.0625, 13.5] in log t, reweighted towards equal relative
//      errors (2.6e-8).
// The rms errors of h and a against 64 bits are below those of erff and expf on every range of z (|z| < 1/2:
// 3.9e-9 .. 7.1e-9 and 1.3e-8 .. 2.5e-8 against 4.4e-9 .. 7.4e-9 and 1.4e-8 .. 2.6e-8), and the left tail keeps
// its relative accuracy (1e-6 at -5), where 1 + erf cancels.
// bf16 tensors (8 significant bits) use the three-term rational erfc of Abramowitz &
// Stegun 7.1.25 (absolute error of the normal cdf below 1.1e-5, i.e. 1/350 of a bf16
// rounding step at 1) with one exponential shared with the density and all scale
// factors folded into the constants: this epilogue is bound by vector-ALU issue
// (two transcendentals at quarter rate plus 13 other instructions per element).
template <bool FAST, int ACT>
__device__ __forceinline__ void act_both(float z, float& h, float& a) {
    if constexpr (ACT == MOE_RELU) {
        h = fmaxf(z, 0.0f);
        a = z > 0.0f ? 1.0f : 0.0f;
        return;
    }
    if constexpr (!FAST) {
        // lowest power first
        constexpr float CENTRE[6] = {0.39894229f, -0.066490486f, 0.0099737411f, -0.0011868734f, 0.00011374246f, -7.6692668e-06f};
        constexpr float MILLS_NUM[4] = {1.2527357f, 1.0029950f, 0.36051896f, 0.061547495f};
        constexpr float MILLS_DEN[5] = {1.0f, 1.5959138f, 1.0661000f, 0.36044064f, 0.061549164f};
        constexpr float LH = -0.72134751f;                             // -log2(e) / 2
        constexpr float PHI0 = 0.39894228f, PHI0_LN2 = 0.27652571f;    // 1 / sqrt(2 pi), times ln 2
        const float t = fminf(fabsf(z), 16.0f), s = t * t;             // phi is 0 from 16 on, also for an infinite z
        const float e = s * LH;
        const float rest = fmaf(s, LH, -e);                            // exp2(e + rest) = exp2(e) (1 + rest ln 2)
        const float pdf = __builtin_amdgcn_exp2f(e) * fmaf(rest, PHI0_LN2, PHI0);
        float c = CENTRE[5], num = MILLS_NUM[3], den = MILLS_DEN[4];
#pragma unroll
        for (int i = 4; i >= 0; --i) c = fmaf(c, s, CENTRE[i]);
#pragma unroll
        for (int i = 2; i >= 0; --i) num = fmaf(num, t, MILLS_NUM[i]);
#pragma unroll
        for (int i = 3; i >= 0; --i) den = fmaf(den, t, MILLS_DEN[i]);
        const float q = num * pdf * __builtin_amdgcn_rcpf(den);
        const float cdf = t < 1.0625f ? fmaf(z, c, 0.5f) : (z >= 0.0f ? 1.0f - q : q);
        h = z * cdf;
        a = fmaf(z, pdf, cdf);
    } else {
        // phi(z) = exp2(-z^2 log2(e)/2 - log2 sqrt(2 pi));  t = 1 / (1 + 0.47047 |z| / sqrt 2)
        const float pdf = __builtin_amdgcn_exp2f(fmaf(z * z, -0.72134752044448170368f, -1.32574806473615920f));
        const float t = __builtin_amdgcn_rcpf(fmaf(0.33267252734483500f, fabsf(z), 1.0f));
        // Phi(-|z|) = erfc(|z|/sqrt 2)/2 = phi(z) t (b1 + b2 t + b3 t^2), b = sqrt(pi/2) (0.3480242, -0.0958798, 0.7478556)
        const float q = t * fmaf(fmaf(0.93729799615056560f, t, -0.12016750882298269f), t, 0.43618364998791710f) * pdf;
        const float cdf = z >= 0.0f ? 1.0f - q : q;
        h = z * cdf;
        a = cdf + z * pdf;
    }
}

// Output of one tile: raw buffer descriptors over the expert's rows in use, so that
// rows >= m_lim fall outside the range and their stores are dropped (no branches).
struct TileOut {
    __amdgpu_buffer_rsrc_t o0, o1, ax;
};

// One row vector of the output tile: off = byte offset inside the expert's output
// (BUF_OOB for a column beyond N), o = element index in the whole tensor (for the
// dropout noise), v = 4 accumulators, aux = the 4 saved derivatives (EPI_MUL only).
template <typename T, int EPI, int ACT>
__device__ __forceinline__ void epilogue4(const GemmArgs& p, const TileOut& to, uint32_t off, size_t o,
                                          float (&v)[4], typename Vec4io<T>::raw aux) {
    if constexpr (EPI == EPI_STORE) {
        Vec4buf<T>::store(to.o0, off, Vec4io<T>::pack(v));
    } else if constexpr (EPI == EPI_H_DACT) {
        float h[4], a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) act_both<sizeof(T) == 2, ACT>(v[i], h[i], a[i]);
        if (p.drop_thr) {   // expert dropout (Sec. 5.4): o is the element index in [E, C, d_ff], a multiple of 4
            uint32_t w[4];
            noise_words(o, MOE_STREAM_DROPOUT, p.seed, w);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float sc = w[i] >= p.drop_thr ? p.drop_scale : 0.0f;
                h[i] *= sc;     // the mask rides in the saved derivative too, so the
                a[i] *= sc;     // backward needs no knowledge of it
            }
        }
        Vec4buf<T>::store(to.o0, off, Vec4io<T>::pack(a));
        Vec4buf<T>::store(to.o1, off, Vec4io<T>::pack(h));
    } else if constexpr (EPI == EPI_H) {
        float h[4], a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) act_both<sizeof(T) == 2, ACT>(v[i], h[i], a[i]);   // the derivative is dead code here
        Vec4buf<T>::store(to.o0, off, Vec4io<T>::pack(h));
    } else if constexpr (EPI == EPI_MUL) {
        float a[4];
        Vec4io<T>::unpack(aux, a);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] *= a[i];
        Vec4buf<T>::store(to.o0, off, Vec4io<T>::pack(v));
    } else {
        Vec4buf<float>::store(to.o0, off, make_float4(v[0], v[1], v[2], v[3]));
    }
}

// The large-tile kernel (bf16).  NWN = wavefronts along N; 2 along M.
template <int BM, int BN, int BK, bool A_KC, bool B_KC, int NWN>
struct GemmSmem {
    typedef bf16_t T;
    static constexpr int NT = 128 * NWN;        // threads per workgroup
    typedef Tile<T, BM, BK, A_KC, NT> TA;
    typedef Tile<T, BN, BK, B_KC, NT> TB;
    static constexpr int STAGE = TA::BYTES + TB::BYTES;
    // LDS ring: one slab being multiplied, one in flight (as many as fit beside the epilogue strips)
    static constexpr int NSTAGE = 2;
    static constexpr int EPI_LD = BN / NWN + 8; // floats per staged epilogue row (4 rows apart -> other bank half)
    static constexpr int EPI_ROWS = 8;          // one accumulator register quad of both lane halves
    static constexpr size_t RING = (size_t)NSTAGE * STAGE;
    static constexpr size_t EPILOGUE = 2 * NWN * EPI_ROWS * (size_t)EPI_LD * sizeof(float);  // wave-private strips
    static constexpr size_t BYTES = RING + EPILOGUE;   // the epilogue never touches the ring
    static constexpr int LOADS = TA::PER_THREAD + TB::PER_THREAD;  // per thread per slab
    static_assert(NSTAGE * LOADS < 64, "vmcnt is a 6-bit counter");
    static_assert((BK / Mma<T>::KSTEP) % 2 == 0, "fragment double buffering needs an even number of k-steps");
    static_assert(BYTES + 4096 <= 160 * 1024, "LDS of one CU (the tile-walk table follows)");
};

// inclusive sums over the lanes of a wave, without LDS
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);     // row_shr 1, 2, 4, 8: inside rows of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);    // row_bcast 15: rows 0 and 2 into the next ones
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);    // row_bcast 31: the lower half into the upper
    return v;
}
// the largest value of a wave's lanes (0 or more)
__device__ __forceinline__ int wave_max_scan(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// The walk of one workgroup over its tiles.  Only tiles that hold rows exist:
// expert e has ceil(n_e / BM) row tiles (all of them if the expert count is the
// reduction length: an empty expert's weight gradient is still written, as zeros).
// A table in LDS holds the running number of tiles per expert.  The tile
// sequence (expert-major) is dealt block-cyclically: with S workgroups per XCD
// (workgroup w serves XCD w % 8: ids are dealt round-robin to the XCDs), block b
// of S consecutive tiles goes to XCD b % 8, one tile per workgroup.  The tiles an
// XCD works on at one time are neighbours and share operand panels in its L2;
// every workgroup gets the same number of tiles up to one (but for a launch's second
// product: follow()); and the tiles of a heavily loaded expert (long reductions in the
// weight-gradient GEMMs) are spread over all workgroups instead of piling up on one XCD.
#define TILE_EPILOGUE 300               // a tile's time: its reduction, and about this many entries' worth of epilogue
#define WALK_BAND 4                     // row tiles per band of the walk inside an expert
#define WALK_CNT 260                    // the experts' row counts follow the 257 running tile counts
#define WALK_BYTES ((WALK_CNT + 256) * 4)
template <int BM, int BN>
struct TileWalk {
    const int* tp;          // LDS: tiles before expert e (tp[256] = all tiles)
    // Smaller tiles and at most 64 experts: lane e holds its expert's rows and the tiles up to its last one, and no LDS
    // or barrier is needed (0.9 us less at the start of a launch).
    bool in_regs = false;
    int rn, rt;
    int ahead = 0, rest = 0;           // rounds that only `rest` of the workgroups take, first
    int t, t_end, step;
    int e, m0, n0, m_lim, k_lim;   // current tile

    // Fills the table (wave 0; 4 experts per lane) and synchronises the workgroup.
    __device__ static __forceinline__ void build(const GemmArgs& p, unsigned char* lds) {
        int* tpw = reinterpret_cast<int*>(lds);
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            int a[4];
            int sa = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ex = 4 * lane + i;
                int n = ex < p.E ? p.expert_count[ex] : 0;
                n = max(0, min(n, p.var_k ? p.K : p.M));
                tpw[WALK_CNT + ex] = n;
                const int tm = ex >= p.E ? 0 : (p.var_k ? p.tiles_m : (n + BM - 1) / BM);
                a[i] = tm * p.tiles_n;
                sa += a[i];
            }
            int ia = sa;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int va = __shfl_up(ia, o, MOE_WAVE);
                if (lane >= o) ia += va;
            }
            int ea = ia - sa;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                tpw[4 * lane + i] = ea;
                ea += a[i];
            }
            if (lane == 63) tpw[256] = ea;
        }
        __syncthreads();
    }
    // `more` = tiles of the launch's later product.  A grid larger than the number of tiles still
    // spreads them over all XCDs.
    __device__ __forceinline__ void start(const GemmArgs& p, const unsigned char* lds, int more) {
        tp = reinterpret_cast<const int*>(lds);
        t_end = __builtin_amdgcn_readfirstlane(tp[256]);
        const int S = min((int)(gridDim.x >> 3), (t_end + more + 7) / 8);
        step = 8 * S;
        t = place() - step;
    }
    // the workgroup's place among the `step` that take turns
    __device__ __forceinline__ int place() const {
        const int i = (int)(blockIdx.x >> 3);
        return i < step >> 3 ? (int)(blockIdx.x & 7) * (step >> 3) + i : 0x3fffffff;
    }
    // The walk over the launch's second product goes on where the first one's ended: it needs the number of workgroups
    // that take turns and of the first product's tiles.
    struct Where { int step, total; };
    __device__ __forceinline__ Where where() const { return {step, t_end}; }
    __device__ __forceinline__ void resume(const GemmArgs& p, Where u, const unsigned char* lds) {
        tp = reinterpret_cast<const int*>(lds);
        t_end = __builtin_amdgcn_readfirstlane(tp[256]);
        step = u.step;
        int most = 0;
        for (int c = 0; c < 256; c += 64) most = max(most, tp[WALK_CNT + c + (threadIdx.x & 63)]);
        follow(u.total, p.lead, wave_max_scan(most));
    }
    // The second product's tiles (t_end of them), after `total` of the first were dealt one by one.  Workgroups that got
    // none in the first product's last round take `rounds` of the second's before all take turns again: as many as such a
    // tile lasts, so that a long one (thousands of reduction entries in dxd) does not bring its workgroup a full share of
    // the others on top.  dxd with dW1 for 7 experts of 470 rows, d = 1720, f = 5520: 258 -> 219 us; 11 of 171,
    // d = 1560, f = 5168: 259 -> 226; 512 tokens on 8 experts, d = 512, f = 2048 (64 x 64): 24.5 -> 20.2.  Counted by the
    // expert with the most rows (`most`: the longest tiles of the second product): by the rows to be expected, a hot expert's
    // were dealt two and three to a workgroup (11 experts, 14288 rows, Zipf gate, d = 1920, f = 2264: 631 us dealt evenly, 667).  The other
    // experts' are shorter, so an eighth of a tile over a whole number counts as one more (14 experts of 14 rows, one of them
    // 48, d = 368, f = 1424, 1.92 tiles: backward 85.7 us with two rounds, 81.0 with three; 41 experts, Zipf gate, 250 rows,
    // d = 664, f = 768 194.9 and 187.3; 29 of 538, d = 304, f = 448 42.0 and 43.6).
    __device__ __forceinline__ void follow(int total, int lead, int most) {
        const int late = total - quotient(total, step) * step, at = place(), tile = most + TILE_EPILOGUE;
        const int rounds = quotient(lead + tile + (tile >> 3) - 1, tile);
        rest = step - late;
        ahead = late > 0 && at >= late ? rounds : 0;
        // one tile every `rest`, then one every `step`: the step between the two is a whole one
        t = ahead > 0 ? at - late - rest : (late > 0 ? rounds * rest : 0) + at - step;
    }
    __device__ __forceinline__ void count(const GemmArgs& p) {
        in_regs = true;
        const int lane = threadIdx.x & 63;
        rn = lane < p.E ? p.expert_count[lane] : 0;
        rn = max(0, min(rn, p.var_k ? p.K : p.M));
        rt = lane >= p.E ? 0 : (p.var_k ? p.tiles_m : (rn + BM - 1) / BM) * p.tiles_n;
        rt = wave_scan(rt);
        t_end = __builtin_amdgcn_readlane(rt, 63);
    }
    // The workgroup's first tile: as start(), but where the tiles of both products of a launch fit in one round, an XCD
    // has its share of each.  `other` = tiles of the other product, `second`: this is the later one.  Also where there are
    // more tiles than CUs: one product after the other, the first one's are some XCDs' alone (13 experts of 62 rows, d = 376,
    // f = 504, 728 tiles of 64 x 64: both launches 22.1 us, 14.4 side by side; 5 of 232, d = 504, f = 2016 43.9 and 39.0).  Where
    // the second product's tiles last many times as long and share CUs with the first's, it can cost (15702 rows, Zipf gate,
    // d = f = 256, 274 tiles: one launch 61 us in a row, 64 side by side).
    __device__ __forceinline__ void begin(const GemmArgs& p, int other, bool second) {
        const int xcd = (int)(blockIdx.x & 7), i = (int)(blockIdx.x >> 3), G = (int)(gridDim.x >> 3);
        const int S = (t_end + 7) >> 3, O = (other + 7) >> 3;
        if (S + O <= G) {
            const int j = second ? i - O : i;
            step = 0x3fffffff;
            t = (j >= 0 && j < S ? xcd * S + j : t_end) - step;
        } else {
            step = 8 * min(G, (t_end + other + 7) >> 3);
            if (second) follow(other, p.lead, wave_max_scan(rn)); else t = place() - step;
        }
    }
    // Inside an expert the tiles are taken band by band: a band is WALK_BAND row tiles high and all column tiles wide, and
    // inside it the row tile varies fastest.  A run of 32 consecutive tiles (what one XCD works on at a time) is then a
    // 4 x 8 block that shares 4 + 8 operand panels in the XCD's L2, whatever the expert's size (one row tile per column
    // tile, or the reverse, would fetch 32 + 1 panels for the same 32 tiles; one expert of 2494 rows, d = 408, f = 376,
    // forward: 15.0 us with the row tile fastest over all of them).
    __device__ __forceinline__ void place_in_expert(int rem, int tiles_m, int tiles_n) {
        const int band = quotient(rem, WALK_BAND * tiles_n);
        const int r = rem - band * WALK_BAND * tiles_n;
        const int rows = min(WALK_BAND, tiles_m - band * WALK_BAND);   // the last band may be lower
        const int tn = quotient(r, rows);
        m0 = (band * WALK_BAND + (r - tn * rows)) * BM;
        n0 = tn * BN;
    }
    // One tile per workgroup, as set_direct() numbered them: nothing waits for the expert's row count but what needs it (a
    // scalar load).  Each XCD has an eighth of each product's tiles.
    __device__ __forceinline__ bool only(const GemmArgs& p) {
        t = t_end = step = 0;
        const int xcd = (int)(blockIdx.x & 7), j = (int)(blockIdx.x >> 3) - p.direct_first;
        const int S = (p.direct_count + 7) >> 3, i = xcd * S + j;
        if (j < 0 || j >= S || i >= p.direct_count) return false;
        e = p.inv_expert ? (int)__umulhi((uint32_t)i, p.inv_expert) : i;
        const int rem = i - e * p.tiles_m * p.tiles_n;
        if (p.tiles_m <= WALK_BAND) {       // one band, found sooner (0.5 us of a 6 us product)
            const int tn = p.inv_m ? (int)__umulhi((uint32_t)rem, p.inv_m) : rem;
            m0 = (rem - tn * p.tiles_m) * BM;
            n0 = tn * BN;
        } else {
            place_in_expert(rem, p.tiles_m, p.tiles_n);
        }
        const int n_e = *((const __attribute__((address_space(4))) int32_t*)(uintptr_t)p.expert_count + e);
        m_lim = p.var_k ? p.M : n_e;
        k_lim = p.var_k ? max(0, min(n_e, p.K)) : p.K;
        return true;
    }
    // only()'s rows, now that B's first loads are on their way; does the tile hold any
    __device__ __forceinline__ bool arrived(const GemmArgs& p) {
        asm volatile("" : "+s"(m_lim));
        m_lim = max(0, min(m_lim, p.M));
        return m0 < m_lim;
    }
    // a / d for a >= 0 and quotients below 2^22: the estimate is at most one off
    __device__ static __forceinline__ int quotient(int a, int d) {
        const int q = __builtin_amdgcn_readfirstlane((int)((float)a * __builtin_amdgcn_rcpf((float)d)));
        const int r = a - q * d;
        return q + (r >= d) - (r < 0);
    }
    // moves to the workgroup's next tile; false when the walk is over
    __device__ __forceinline__ bool next(const GemmArgs& p) {
        t += ahead > 0 ? rest : step;
        --ahead;
        if (t >= t_end) return false;
        // the expert that owns tile t: as many experts end at or before it
        int first, n_e;
        if (in_regs) {
            e = __popcll(__ballot(rt <= t));
            n_e = __builtin_amdgcn_readlane(rn, e);
            first = __builtin_amdgcn_readlane(rt, e) - (p.var_k ? p.tiles_m : (n_e + BM - 1) / BM) * p.tiles_n;
        } else {
            e = 0;
            for (int c = 0; c < p.E; c += 64) e += __popcll(__ballot(tp[c + (threadIdx.x & 63) + 1] <= t));
            // everything here is the same in every lane; keep it in scalar registers
            e = __builtin_amdgcn_readfirstlane(e);
            first = __builtin_amdgcn_readfirstlane(tp[e]);
            n_e = __builtin_amdgcn_readfirstlane(tp[WALK_CNT + e]);
        }
        const int rem = t - first;
        const int tm_e = p.var_k ? p.tiles_m : (n_e + BM - 1) / BM;   // row tiles of this expert
        place_in_expert(rem, tm_e, p.tiles_n);
        m_lim = p.var_k ? p.M : n_e;
        k_lim = p.var_k ? n_e : p.K;
        return true;
    }
};

// Persistent workgroups: each walks its tiles and treats the slabs of all of
// them as one stream through the LDS ring, so the first slabs of the next tile
// are already resident when the epilogue of the current one ends, and no
// workgroup launch or cold first load sits between two tiles.
template <int BM, int BN, int BK, bool A_KC, bool B_KC, int EPI, int ACT, int NWN, bool KG>
__device__ __forceinline__ typename TileWalk<BM, BN>::Where gemm_body(const GemmArgs& p, int more, typename TileWalk<BM, BN>::Where before) {
    typedef bf16_t T;
    typedef GemmSmem<BM, BN, BK, A_KC, B_KC, NWN> SM;
    typedef typename SM::TA TA;
    typedef typename SM::TB TB;
    typedef typename Vec4io<T>::raw raw;
    constexpr int TM = BM / 64, TN = BN / (32 * NWN);  // 32x32 MFMA tiles per wave (2 x NWN waves)
    constexpr int KS = BK / Mma<T>::KSTEP;
    constexpr int NS = SM::NSTAGE;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / NWN, wn = wave % NWN;
    const int l32 = lane & 31, g = lane >> 5;

    // epilogue geometry: the wave's (BM/2) x (BN/2) sub-tile leaves in strips of 8
    // rows; a lane owns 4 consecutive columns of RPI-strided rows
    constexpr int ELD = SM::EPI_LD;
    constexpr int WCOLS = BN / NWN;
    constexpr int LPR = WCOLS / 4;                // lanes per staged row
    constexpr int RPI = 64 / LPR;                 // rows per wave instruction
    constexpr int NIT = SM::EPI_ROWS / RPI;       // row vectors per lane per strip
    static_assert(NIT >= 1, "strip narrower than a wavefront");
    const int er = lane / LPR, ec = (lane - er * LPR) * 4;
    float* strip = reinterpret_cast<float*>(smem_raw + SM::RING) + wave * SM::EPI_ROWS * ELD;

    // ---- producer: the stream of slabs of all tiles of this workgroup ---------
    unsigned char* walk_lds = smem_raw + SM::BYTES;
    TileWalk<BM, BN>::build(p, walk_lds);
    TileWalk<BM, BN> pw;       // tile whose slabs are being requested
    if (more < 0) pw.resume(p, before, walk_lds); else pw.start(p, walk_lds, more);
    bool p_more = pw.next(p);
    int p_kt = 0, p_nk = 0;
    u32x4_t dsA = {0, 0, 0, 0}, dsB = {0, 0, 0, 0};
    typename TA::Plan planA;
    typename TB::Plan planB;
    auto producer_setup = [&]() {
        dsA = TA::desc((const T*)p.A + (size_t)pw.e * p.strideA, p.lda, pw.m_lim, pw.k_lim);
        dsB = TB::desc((const T*)p.B + (size_t)pw.e * p.strideB, p.ldb, p.N, pw.k_lim);
        TA::plan(planA, p.lda, pw.m0, pw.m_lim);
        TB::plan(planB, p.ldb, pw.n0, p.N);
        p_kt = 0;
        p_nk = (pw.k_lim + BK - 1) / BK;
    };
    if (p_more) producer_setup();
    // requests the next slab of the stream into ring stage `st`; past the end of
    // the stream it requests out-of-range loads (zeros) so that every slab counts
    // the same number of loads in vmcnt
    // The request of a slab is split in two so that, inside the main loop, its
    // loads can be issued one at a time between MFMAs (a burst of all of them fills
    // the address FIFO of the memory pipe and stalls the wave's instruction issue).
    int pk0 = 0, pkl = 0;
    uint32_t plds = 0;
    u32x4_t pua = {0, 0, 0, 0}, pub = {0, 0, 0, 0};
    auto produce_prepare = [&](int st) {
        while (p_more && p_kt >= p_nk) {
            p_more = pw.next(p);
            if (p_more) producer_setup();
        }
        pk0 = p_more ? p_kt * BK : 0;
        pkl = p_more ? pw.k_lim : 0;              // k_lim 0: every guard fails, nothing is read
        if (!p_more) { dsA[2] = 0; dsB[2] = 0; }  // empty range: every load returns zeros
        const u32x4_t sdA = TA::slab_desc(dsA, TA::slab_shift(p.lda, pk0)), sdB = TB::slab_desc(dsB, TB::slab_shift(p.ldb, pk0));
        // the descriptors are wave-uniform by construction; say so to the compiler
        // (they must sit in scalar registers for the load instruction)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pua[i] = __builtin_amdgcn_readfirstlane(sdA[i]);
            pub[i] = __builtin_amdgcn_readfirstlane(sdB[i]);
        }
        plds = lds0 + st * SM::STAGE;
        ++p_kt;
    };
    auto produce_issue = [&](int i) {   // load i of the prepared slab (i < SM::LOADS; A's loads come first)
        if (i < TA::PER_THREAD) TA::template issue_one<KG>(planA, pua, pk0, pkl, plds, i);
        else TB::template issue_one<KG>(planB, pub, pk0, pkl, plds + TA::BYTES, i - TA::PER_THREAD);
    };
    auto produce = [&](int st) {
        produce_prepare(st);
#pragma unroll
        for (int i = 0; i < SM::LOADS; ++i) produce_issue(i);
    };

    // ---- consumer ---------------------------------------------------------------
    TileWalk<BM, BN> cw;
    if (more < 0) cw.resume(p, before, walk_lds); else cw.start(p, walk_lds, more);
    if (!cw.next(p)) return cw.where();    // nothing to do for this workgroup (uniform)
#pragma unroll
    for (int s = 0; s < NS; ++s) produce(s);
    // slab 0 of the stream has landed once at most the NS-1 younger slabs are outstanding
    wait_vmcnt<(NS - 1) * SM::LOADS>();
    __syncthreads();
    // Two-stage ring with four k-steps per slab: the B half of a stage is released
    // early.  A wave needs few B fragments (TN per k-step), so it reads those of all four k-steps
    // during the slab's first step; one barrier later nobody reads the B half again and it is
    // refilled three k-steps before the A half.  The two halves of a slab are then requested at
    // different times, there is (almost) always a request in flight, and B has 1.75 slab periods
    // to arrive instead of one.
    // (not in the instance whose epilogue keeps saved-derivative rows in registers through the
    // main loop: the extra fragment registers would spill there)
    static_assert(NS == 2 && KS == 4, "the schedules below are laid out by hand for these");
    constexpr bool BEARLY = EPI != EPI_MUL;
    typename Mma<T>::frag fa[2][TM], fb[BEARLY ? KS : 2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = TA::frag(smem_raw, wm * (BM / 2) + i * 32, 0, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = TB::frag(smem_raw + TA::BYTES, wn * WCOLS + j * 32, 0, lane);
    int stage = 0;

    bool again = true;
    while (again) {
        const int nk = (cw.k_lim + BK - 1) / BK;
        const size_t obase = (size_t)cw.e * p.strideO;
        const int ncol = cw.n0 + wn * WCOLS + ec;
        const int mrow = cw.m0 + wm * (BM / 2) + er;
        const int m_lim = cw.m_lim;

        // EPI_MUL: the saved derivative does not depend on the product.  The rows of
        // the first two 32-row blocks are requested now and ride in registers through
        // the main loop; the later blocks are requested while earlier ones are written.
        constexpr int AUXB = EPI == EPI_MUL ? 2 : 1;
        raw aux[AUXB][EPI == EPI_MUL ? 4 : 1][EPI == EPI_MUL ? NIT : 1];
        constexpr uint32_t OSZ = EPI == EPI_F32 ? 4u : (uint32_t)sizeof(T);   // bytes per output element
        const size_t obytes = (size_t)m_lim * p.ldo * OSZ;                    // the expert's rows in use
        TileOut to;
        to.o0 = buf_rsrc((const char*)p.out0 + obase * OSZ, obytes);
        to.o1 = buf_rsrc(EPI == EPI_H_DACT ? (const char*)p.out1 + obase * OSZ : nullptr, EPI == EPI_H_DACT ? obytes : 0);
        to.ax = buf_rsrc(EPI == EPI_MUL ? (const char*)p.aux + obase * OSZ : nullptr, EPI == EPI_MUL ? obytes : 0);
        const bool col_ok = ncol < p.N;
        // byte offset of this lane's row vector in row m of the expert's output; a row
        // >= m_lim lies beyond the descriptor's range by itself
        auto out_off = [&](int m) { return col_ok ? (uint32_t)(((size_t)m * p.ldo + ncol) * OSZ) : BUF_OOB; };
        auto fetch_aux = [&](int buf, int i) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int it = 0; it < NIT; ++it)
                    aux[buf][q][it] = Vec4buf<T>::load(to.ax, out_off(mrow + i * 32 + q * 8 + it * RPI));
        };
        if constexpr (EPI == EPI_MUL) {
            if (nk == 0) {
#pragma unroll
                for (int i = 0; i < AUXB; ++i) fetch_aux(i, i);
            }
        }

        f32x16_t acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

        for (int kt = 0; kt < nk; ++kt) {
            const unsigned char* a_s = smem_raw + stage * SM::STAGE;
            const unsigned char* b_s = a_s + TA::BYTES;
            const int next = stage == NS - 1 ? 0 : stage + 1;
            if constexpr (BEARLY) {
                constexpr int NMMA = TM * TN;
                static_assert(NMMA == 2 * TM && TN <= TM && NMMA % TB::PER_THREAD == 0 && NMMA % TA::PER_THREAD == 0, "slots of the requests and fragment reads below");
                // ---- k-step 0: MFMAs on (fa[0], fb[0]); A fragments of step 1 and B fragments of steps 1..3
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[1][i] = TA::frag(a_s, wm * (BM / 2) + i * 32, 1, lane);
#pragma unroll
                for (int ks = 1; ks < KS; ++ks)
#pragma unroll
                    for (int j = 0; j < TN; ++j) fb[ks][j] = TB::frag(b_s, wn * WCOLS + j * 32, ks, lane);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::mma(fa[0][i], fb[0][j], acc[i][j]);
#pragma unroll
                for (int q = 0; q < NMMA; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);   // LDS reads
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                }
                __builtin_amdgcn_sched_barrier(0);
                // every B fragment of this slab is in registers once this wave's LDS reads have
                // returned; when all waves are here the B half of the stage is refilled
                wait_vmcnt_lgkm0<63>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                produce_prepare(stage);
                // ---- k-step 1: MFMAs on (fa[1], fb[1]); B requests; A fragments of step 2
                // (a wave issues its instructions strictly one after another, an MFMA holding it for the
                // MFMA's 32 cycles: only the other wave of the SIMD can fill the matrix pipe meanwhile.  The
                // requests and fragment reads are therefore dealt evenly over the MFMA slots - a long run of
                // them in one place leaves the pipe idle whenever both waves are in such a run.)
#pragma unroll
                for (int q = 0; q < NMMA; ++q) {
                    constexpr int LSTEP = NMMA / TB::PER_THREAD;   // a request every LSTEP slots
                    if (q % LSTEP == 0) produce_issue(TA::PER_THREAD + q / LSTEP);
                    if (q % 2 == 1) fa[0][q / 2] = TA::frag(a_s, wm * (BM / 2) + q / 2 * 32, 2, lane);
                    acc[q / TN][q % TN] = Mma<T>::mma(fa[1][q / TN], fb[1][q % TN], acc[q / TN][q % TN]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // ---- k-step 2: MFMAs on (fa[0], fb[2]); A fragments of step 3
#pragma unroll
                for (int q = 0; q < NMMA; ++q) {
                    if (q % 2 == 0) fa[1][q / 2] = TA::frag(a_s, wm * (BM / 2) + q / 2 * 32, 3, lane);
                    acc[q / TN][q % TN] = Mma<T>::mma(fa[0][q / TN], fb[2][q % TN], acc[q / TN][q % TN]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // ---- k-step 3: the next slab (requested a slab period ago for A, 1.75 for B) has
                // landed once only the B requests of this slab's step 1 are outstanding (loads complete
                // in order; anything else that is younger only makes the wait longer); every A
                // fragment of this slab is in registers, so the A half is refilled; the next
                // slab's first fragments are fetched under the MFMAs on (fa[1], fb[3])
                wait_vmcnt_lgkm0<TB::PER_THREAD>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if constexpr (EPI == EPI_MUL) {
                    if (kt == 0) {
#pragma unroll
                        for (int i = 0; i < AUXB; ++i) fetch_aux(i, i);
                    }
                }
                const unsigned char* a_n = smem_raw + next * SM::STAGE;
#pragma unroll
                for (int q = 0; q < NMMA; ++q) {
                    constexpr int LSTEP = NMMA / TA::PER_THREAD;
                    if (q % LSTEP == 0) produce_issue(q / LSTEP);
                    // odd slots: one A fragment each; the B fragments (needed first) ride with the first ones
                    if (q % 2 == 1) {
                        const int i = q / 2;
                        fa[0][i] = TA::frag(a_n, wm * (BM / 2) + i * 32, 0, lane);
                        if (i < TN) fb[0][i] = TB::frag(a_n + TA::BYTES, wn * WCOLS + i * 32, 0, lane);
                    }
                    acc[q / TN][q % TN] = Mma<T>::mma(fa[1][q / TN], fb[3][q % TN], acc[q / TN][q % TN]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                stage = next;
                continue;
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int c = ks & 1, n = c ^ 1;   // KS is even: every slab starts in buffer 0
                if (ks + 1 < KS) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[n][i] = TA::frag(a_s, wm * (BM / 2) + i * 32, ks + 1, lane);
#pragma unroll
                    for (int j = 0; j < TN; ++j) fb[n][j] = TB::frag(b_s, wn * WCOLS + j * 32, ks + 1, lane);
                } else {
                    // Before the last k-step of a slab: its fragments are already in
                    // registers (requested one step ago; the wait below covers them), so once
                    // every wave is here nobody reads this stage again and it is refilled at
                    // once with the slab NS positions down the stream.  The next slab (this
                    // tile's or the next tile's first) has landed once at most the NS-2
                    // younger ones are outstanding; its first fragments are fetched under
                    // this slab's last MFMAs.
                    wait_vmcnt_lgkm0<(NS - 2) * SM::LOADS>();
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    if constexpr (EPI == EPI_MUL) {
                        // requested right after a wait, a whole slab period before the next one:
                        // every wait of the loop is for all outstanding loads, these included
                        if (kt == 0) {
#pragma unroll
                            for (int i = 0; i < AUXB; ++i) fetch_aux(i, i);
                        }
                    }
                    produce_prepare(stage);
                    const unsigned char* a_n = smem_raw + next * SM::STAGE;
                    // hand-laid schedule of the last step: per MFMA one slab request and one
                    // fragment read of the next slab
                    constexpr int NMMA = TM * TN, LPM = (SM::LOADS + NMMA - 1) / NMMA;
#pragma unroll
                    for (int q = 0; q < NMMA; ++q) {
#pragma unroll
                        for (int u = 0; u < LPM; ++u)
                            if (q * LPM + u < SM::LOADS) produce_issue(q * LPM + u);
                        if (q < TM) fa[n][q] = TA::frag(a_n, wm * (BM / 2) + q * 32, 0, lane);
                        else if (q < TM + TN) fb[n][q - TM] = TB::frag(a_n + TA::BYTES, wn * WCOLS + (q - TM) * 32, 0, lane);
                        acc[q / TN][q % TN] = Mma<T>::mma(fa[c][q / TN], fb[c][q % TN], acc[q / TN][q % TN]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    static_assert(TM + TN <= NMMA, "one fragment read per MFMA slot");
                    continue;
                }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::mma(fa[c][i], fb[c][j], acc[i][j]);
                // issue order: the fragment reads of the next k-step go out under the
                // first MFMAs of this one, so a full step of matrix work covers their latency
#pragma unroll
                for (int q = 0; q < TM * TN; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // LDS reads
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                }
                __builtin_amdgcn_sched_barrier(0);   // no MFMA drifts into the next step
            }
            stage = next;
        }

        // ---- epilogue: accumulators -> wave-private LDS strip -> row vectors --------
        // accumulator element v of lane l in a 32x32 tile: column l%32,
        // row 8*(v/4) + 4*(l/32) + v%4; strip s = (i, q) = (s/4, s%4) holds rows i*32 + 8q .. +7.
        // LDS operations of a wave execute in order, so strip s+1 is written and read
        // back (into the other register set) before the vectors of strip s are used:
        // the LDS round trip of every strip hides behind the previous strip's work.
        constexpr int NSTRIP = 4 * TM;
        const int rows_left = __builtin_amdgcn_readfirstlane(m_lim - cw.m0 - wm * (BM / 2));
        auto write_strip = [&](int s_) {
            const int i = s_ >> 2, q = s_ & 3;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) strip[(4 * g + r) * ELD + j * 32 + l32] = acc[i][j][4 * q + r];
        };
        auto read_strip = [&](float4 (&w)[NIT]) {
#pragma unroll
            for (int it = 0; it < NIT; ++it) w[it] = *reinterpret_cast<const float4*>(strip + (er + it * RPI) * ELD + ec);
        };
        constexpr bool ROLLED = EPI == EPI_H_DACT || EPI == EPI_H;   // long per-vector code: kept in a rolled loop
        float4 w[ROLLED ? 1 : 2][NIT];
        write_strip(0);
        if constexpr (!ROLLED) read_strip(w[0]);
#pragma unroll
        for (int s_ = 0; s_ < NSTRIP; ++s_) {
            const int i = s_ >> 2, q = s_ & 3;
            const int m_strip = mrow + i * 32 + q * 8;
            if (ROLLED && q == 0 && i * 32 >= rows_left) break;      // no row in use from here on (uniform)
            if constexpr (ROLLED) {
                // one copy of the activation code per strip; the next vector is read from
                // LDS before the current one is worked on (carried in registers, no arrays)
                float4 cur = *reinterpret_cast<const float4*>(strip + er * ELD + ec);
#pragma unroll 1
                for (int it = 0; it < NIT; ++it) {
                    const int itn = it + 1 < NIT ? it + 1 : it;
                    const float4 nxt = *reinterpret_cast<const float4*>(strip + (er + itn * RPI) * ELD + ec);
                    float v[4] = {cur.x, cur.y, cur.z, cur.w};
                    const int m = m_strip + it * RPI;
                    epilogue4<T, EPI, ACT>(p, to, out_off(m), obase + (size_t)m * p.ldo + ncol, v, Vec4io<T>::zero());
                    cur = nxt;
                }
                if (s_ + 1 < NSTRIP) write_strip(s_ + 1);
            } else {
                if (s_ + 1 < NSTRIP) {
                    write_strip(s_ + 1);
                    read_strip(w[(s_ + 1) & 1]);
                }
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const float4 x4 = w[s_ & 1][it];
                    float v[4] = {x4.x, x4.y, x4.z, x4.w};
                    const int m = m_strip + it * RPI;
                    epilogue4<T, EPI, ACT>(p, to, out_off(m), 0, v,
                                           aux[EPI == EPI_MUL ? i % AUXB : 0][EPI == EPI_MUL ? q : 0][EPI == EPI_MUL ? it : 0]);
                }
            }
            if constexpr (EPI == EPI_MUL) {
                if (q == 3 && i + AUXB < TM) fetch_aux(i % AUXB, i + AUXB);   // the buffer just used is free again
            }
        }
        again = cw.next(p);
    }
    // the zero-fill loads requested past the end of the stream target this
    // workgroup's LDS: wait for them before the workgroup retires
    wait_vmcnt<0>();
    return cw.where();
}

template <int BM, int BN, int BK, bool A_KC, bool B_KC, int EPI, int ACT, int NWN, bool KG>
__global__ __launch_bounds__(128 * NWN, 2) void grouped_gemm_kernel(const GemmArgs p) {   // two waves per SIMD: at most 256 registers
    gemm_body<BM, BN, BK, A_KC, B_KC, EPI, ACT, NWN, KG>(p, 0, {0, 0});
}

// Two independent grouped GEMMs in one launch: every workgroup walks its tiles of the
// first, then its tiles of the second.  Nothing is synchronised between workgroups (the
// two products must not depend on each other), so a workgroup that is done with the first
// starts the second at once: one launch, one ramp-up and one tail instead of two, and the
// workgroups drift apart, which spreads the store bursts of their epilogues.
template <int BM, int BN, int BK, bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2, int NWN, bool KG>
__global__ __launch_bounds__(128 * NWN, 2) void grouped_gemm_pair_kernel(const GemmArgs p1, const GemmArgs p2) {
    const typename TileWalk<BM, BN>::Where w = gemm_body<BM, BN, BK, A1, B1, EPI1, 0, NWN, KG>(p1, p2.E * p2.tiles_m * p2.tiles_n, {0, 0});
    __syncthreads();      // every wave is done with the ring and the tile table of the first product
    gemm_body<BM, BN, BK, A2, B2, EPI2, 0, NWN, KG>(p2, -1, w);
}

// ---------------------------------------------------------------------------
// The same products on smaller tiles (64 x 64 or 128 x 128, 2 x 2 waves; fp32 with few
// tiles: two such groups share one; fp32's smallest: further below), two or three workgroups per CU (one for the
// two-group forms, whose ring takes 96 KB): for problems that give the large tile too few workgroups, for
// experts with few rows (then the weights' stream from HBM is the bound and the
// other workgroups of a CU keep requests in flight while one is in its prologue or
// epilogue), and for all fp32 tensors.
//
// bf16: slabs of 64 through an NS-stage LDS ring, filled by loads that write LDS
// directly; one barrier per slab.
//
// fp32 on the bf16 matrix pipe: every fp32 value is split into three bf16 parts
// rounded to nearest, hi + mid + lo = value exactly (8 significant bits each and the
// signs of the residuals), and a product is the six partial products of weight
// above 2^-26; each is exact in fp32 and all are summed in fp32 by the MFMAs.  The
// parts left out are below a quarter of the rounding error of one fp32 product.  Six
// v_mfma_f32_32x32x16_bf16 (32 cycles each) replace eight v_mfma_f32_32x32x2_f32 (64
// cycles each); results are nearer to the exact ones than the fp32 pipe's (relative
// error of yd at d = 512, f = 2048: 3e-7 against 9e-7).  A slab is split once per
// workgroup on its way from registers to LDS, under the MFMAs of the slab before.  T = 4096,
// d = 512, f = 2048, E = 8, top-2, the four launches: 1033 us on the fp32 pipe, 609 now, with the
// matrix pipe busy in 39 - 51 % of the cycles and vector instructions issued in 28 - 37 %: the
// split of every slab in every workgroup that reads it is what keeps the two apart from the
// 225 us that six partial products take at the pipe's peak.  The parts hold a
// value exactly from 2^-110 to 3.39e38; results that operands outside of that range, or
// infinite or NaN ones, may have reached are formed again on the fp32 pipe (redo_f32).
//
// The products are computed with the operands exchanged (D^T), so that a lane holds four
// consecutive columns of one output row: the epilogue's LDS strip is written and read
// in 16-byte vectors.
// ---------------------------------------------------------------------------
// KW: groups of four waves that share a tile, each taking its part of every slab's k-steps (fp32)
template <typename T, int BM, int BN, int KW, int NS, bool A_KC, bool B_KC>
struct MidSmem {
    static constexpr bool SPLIT = sizeof(T) == 4;
    static constexpr int NT = 256 * KW;
    static constexpr int BK = (SPLIT ? (BM < 128 || BN < 128 ? 32 : 16) : 64) * KW;
    static constexpr int NP = SPLIT ? 3 : 1;               // bf16 planes per operand
    typedef Tile<bf16_t, BM, BK, A_KC, NT> TA;
    typedef Tile<bf16_t, BN, BK, B_KC, NT> TB;
    static constexpr int STAGE = NP * (TA::BYTES + TB::BYTES);
    static_assert(NS >= 2 && (!SPLIT || NS == 2) && (SPLIT || KW == 1), "ring depth and wave groups per path");
    static constexpr int REDUCE = (KW - 1) * BM * BN * 4;
    static constexpr int LOADS = TA::PER_THREAD + TB::PER_THREAD;
    static constexpr int STRIP_LD = BN / 2 + 4;
    static constexpr int STRIPS = 4 * 32 * STRIP_LD * 4;   // the epilogue's strips lie over the ring
    static constexpr int RING = NS * STAGE;
    static constexpr int BYTES = RING > STRIPS ? (RING > REDUCE ? RING : REDUCE) : (STRIPS > REDUCE ? STRIPS : REDUCE);
    // workgroups per CU: what LDS holds, and registers (the fp32 form needs about 180 at 128 x 128)
    static constexpr int FIT = 160 * 1024 / (BYTES + WALK_BYTES);
    static constexpr int OCC = FIT >= 3 && !SPLIT ? 3 : (FIT >= 2 ? 2 : 1);
};

// 8 fp32 of one tile chunk -> three bf16 planes, rounded to nearest at every step: hi + mid + lo = w exactly
// for 2^-110 <= |w| <= 3.39e38.  Below, lo falls under bf16's subnormals; above, hi rounds to infinity and mid
// is then the opposite one, as for an infinite w: every product and sum that such a w enters is NaN or infinite.
__device__ __forceinline__ void split3_rne(const u32x4_t (&w)[2], u32x4_t& hi, u32x4_t& mid, u32x4_t& lo) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = __uint_as_float(w[i >> 1][2 * (i & 1)]), b = __uint_as_float(w[i >> 1][2 * (i & 1) + 1]);
        const uint32_t h = pack_bf16x2(a, b);
        const float a1 = a - __uint_as_float(h << 16), b1 = b - __uint_as_float(h & 0xffff0000u);
        const uint32_t m = pack_bf16x2(a1, b1);
        lo[i] = pack_bf16x2(a1 - __uint_as_float(m << 16), b1 - __uint_as_float(m & 0xffff0000u));
        hi[i] = h;
        mid[i] = m;
    }
}

// May any of this wave's sums hold less than fp32 products would have given?  A sum that is NaN or infinite may
// come from an operand that the split made so; one below 2^-80 that is not zero may come from operands below
// 2^-110 (larger ones in the same sum leave the lost bits, 2^-134 per operand, far below its rounding).
// Rows from `rows` on (this lane's: i * 32 + l32) are not in use and may hold anything.
template <int TM, int TN>
__device__ __forceinline__ bool split_in_doubt(const f32x16_t (&acc)[TM][TN], int rows, int l32) {
    bool doubt = false;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float big[4] = {0.0f, 0.0f, 0.0f, 0.0f};           // four chains: each step waits for the one before; `maximum` keeps NaN
        uint32_t small[4] = {~0u, ~0u, ~0u, ~0u};
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                big[v & 3] = __builtin_elementwise_maximum(big[v & 3], fabsf(acc[i][j][v]));
                small[v & 3] = min(small[v & 3], (__float_as_uint(acc[i][j][v]) << 1) - 1u);      // zeros come out largest
            }
        const bool finite = __builtin_elementwise_maximum(__builtin_elementwise_maximum(big[0], big[1]), __builtin_elementwise_maximum(big[2], big[3])) < INFINITY;
        doubt |= i * 32 + l32 < rows && (!finite || min(min(small[0], small[1]), min(small[2], small[3])) < (127u - 80u) << 24);
    }
    return __ballot(doubt) != 0;
}

// One wave's part of an fp32 tile of expert e on the fp32 pipe, operands straight from memory (m, n: the part's first
// row and column): the exact fallback of the split, for waves that split_in_doubt() sends here.  `args` = which of the
// kernel's arguments describes the product; they are read again here, so that nothing is kept in registers for this.
template <bool A_KC, bool B_KC, int TM, int TN>
__device__ __forceinline__ void redo_f32(f32x16_t (&acc)[TM][TN], int args, int e, int m, int m_lim, int n, int l32, int g) {
    auto base = (const __attribute__((address_space(4))) GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm("" : "+s"(base));
    const __attribute__((address_space(4))) GemmArgs& q = base[args];
    const int lda = q.lda, ldb = q.ldb, N = q.N, k_lim = q.var_k ? max(0, min(q.expert_count[e], q.K)) : q.K;
    const __amdgpu_buffer_rsrc_t rsA = buf_rsrc((const float*)q.A + (size_t)e * q.strideA, (size_t)(A_KC ? m_lim : k_lim) * lda * 4);
    const __amdgpu_buffer_rsrc_t rsB = buf_rsrc((const float*)q.B + (size_t)e * q.strideB, (size_t)(B_KC ? N : k_lim) * ldb * 4);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto load = [&](bool kc, __amdgpu_buffer_rsrc_t rs, int r, int r_lim, int k, int ld) {
        return buf_load_f32(rs, r < r_lim && k < k_lim ? (uint32_t)(kc ? r * ld + k : k * ld + r) * 4u : BUF_OOB);
    };
    constexpr int U = 4;
#pragma unroll 1
    for (int k0 = 0; k0 < k_lim; k0 += 2 * U) {
        float fa[U][TM], fb[U][TN];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[u][i] = load(A_KC, rsA, m + i * 32 + l32, m_lim, k0 + 2 * u + g, lda);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[u][j] = load(B_KC, rsB, n + j * 32 + l32, N, k0 + 2 * u + g, ldb);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[u][j], fa[u][i], acc[i][j], 0, 0, 0);
    }
}

template <typename T, int BM, int BN, int KW, int NS, bool A_KC, bool B_KC, int EPI, int ACT, bool KG>
__device__ __forceinline__ typename TileWalk<BM, BN>::Where mid_body(const GemmArgs& p, int more, typename TileWalk<BM, BN>::Where before) {
    typedef MidSmem<T, BM, BN, KW, NS, A_KC, B_KC> SM;
    typedef typename SM::TA TA;
    typedef typename SM::TB TB;
    constexpr bool SPLIT = SM::SPLIT;
    constexpr int BK = SM::BK, KS = BK / 16 / KW;
    constexpr int TM = BM / 64, TN = BN / 64;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int l32 = lane & 31, g = lane >> 5;
    unsigned char* walk_lds = smem_raw + SM::BYTES;
    TileWalk<BM, BN> w;
    const bool direct = p.direct_count > 0;
    if (direct) {
        if (!w.only(p)) return w.where();
    } else if (p.E <= MOE_WAVE) {
        w.count(p);
        w.begin(p, more < 0 ? before.total : more, more < 0);
    } else {
        TileWalk<BM, BN>::build(p, walk_lds);
        if (more < 0) w.resume(p, before, walk_lds); else w.start(p, walk_lds, more);
    }
    for (bool more_tiles = direct || w.next(p); more_tiles; more_tiles = !direct && w.next(p)) {
        const int nk = (w.k_lim + BK - 1) / BK;
        const T* gA = (const T*)p.A + (size_t)w.e * p.strideA;
        const T* gB = (const T*)p.B + (size_t)w.e * p.strideB;
        if constexpr (EPI == EPI_F32) {
            if (nk == 0) {
                // An expert without rows: its zeros are stored at once.  Through the loop, loads that wait for the
                // stores before them and the barriers would hold back the next tile's (16 empty experts, d = 408,
                // f = 752, fp32 backward: 24.9 -> 17.0 us).
                constexpr int CH = BN / 4;                   // 16-byte pieces of a tile row
                const __amdgpu_buffer_rsrc_t o0 = buf_rsrc((float*)p.out0 + (size_t)w.e * p.strideO, (size_t)w.m_lim * p.ldo * 4);
                const int col = w.n0 + (int)(threadIdx.x % CH) * 4;
                const float zero[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
                for (int row = threadIdx.x / CH; row < BM; row += SM::NT / CH)
                    BufChunk<float>::store(o0, col < p.N ? (uint32_t)((w.m0 + row) * p.ldo + col) * 4u : BUF_OOB, zero);
                continue;
            }
        }
        f32x16_t acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

        bool live;          // does this wave hold any row in use
        if constexpr (!SPLIT) {
            // one operand's part of slab kt, into ring stage st
            auto request_one = [&](auto tile, const auto& plan, u32x4_t ds, int ld, int kt, uint32_t base) {
                typedef decltype(tile) TT;
                const int k0 = kt < nk ? kt * BK : 0;
                u32x4_t sd = TT::slab_desc(ds, TT::slab_shift(ld, k0));
                if (kt >= nk) sd[2] = 0;      // past the end: zeros, so that every slab counts the same loads
#pragma unroll
                for (int i = 0; i < 4; ++i) sd[i] = __builtin_amdgcn_readfirstlane(sd[i]);
#pragma unroll
                for (int i = 0; i < TT::PER_THREAD; ++i) TT::template issue_one<KG>(plan, sd, k0, w.k_lim, base, i);
            };
            typename TB::Plan planB;
            TB::plan(planB, p.ldb, w.n0, p.N);
            const u32x4_t dsB = TB::desc((const bf16_t*)gB, p.ldb, p.N, w.k_lim);
            auto request_b = [&](int kt, int st) { request_one(TB(), planB, dsB, p.ldb, kt, lds0 + st * SM::STAGE + TA::BYTES); };
            request_b(0, 0);                  // B first: A is not touched before the rows in use are known
            if (direct && !w.arrived(p)) {
                wait_vmcnt<0>();
                continue;
            }
            live = w.m0 + wm * (BM / 2) < w.m_lim;
            typename TA::Plan planA;
            TA::plan(planA, p.lda, w.m0, w.m_lim);
            const u32x4_t dsA = TA::desc((const bf16_t*)gA, p.lda, w.m_lim, w.k_lim);
            auto request_a = [&](int kt, int st) { request_one(TA(), planA, dsA, p.lda, kt, lds0 + st * SM::STAGE); };
            request_a(0, 0);
#pragma unroll
            for (int s = 1; s < NS - 1; ++s) {
                request_a(s, s);
                request_b(s, s);
            }
            int st = 0;
            for (int kt = 0; kt < nk; ++kt) {
                wait_vmcnt_lgkm0<(NS - 2) * SM::LOADS>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                request_a(kt + NS - 1, st == 0 ? NS - 1 : st - 1);
                request_b(kt + NS - 1, st == 0 ? NS - 1 : st - 1);
                if (live) {
                    const unsigned char* a_s = smem_raw + st * SM::STAGE;
                    const unsigned char* b_s = a_s + TA::BYTES;
                    // 64 x 64 has one product per k-step: all of the slab's fragments are asked for before the first one.
                    // Left to itself the compiler waited for each k-step's in turn, where it saw more waves to be had
                    // from fewer registers than LDS lets in (h W2, 68 rows, K = 3552: 20.1 us, 18.0 so).
                    constexpr int STEPS = TM * TN == 1 ? KS : 1;
#pragma unroll
                    for (int k0 = 0; k0 < KS; k0 += STEPS) {
                        bf16x8_t fa[STEPS][TM], fb[STEPS][TN];
#pragma unroll
                        for (int ks = 0; ks < STEPS; ++ks) {
#pragma unroll
                            for (int i = 0; i < TM; ++i) fa[ks][i] = TA::frag(a_s, wm * (BM / 2) + i * 32, wk * KS + k0 + ks, lane);
#pragma unroll
                            for (int j = 0; j < TN; ++j) fb[ks][j] = TB::frag(b_s, wn * (BN / 2) + j * 32, wk * KS + k0 + ks, lane);
                        }
                        if (STEPS > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int ks = 0; ks < STEPS; ++ks)
#pragma unroll
                            for (int i = 0; i < TM; ++i)
#pragma unroll
                                for (int j = 0; j < TN; ++j) acc[i][j] = Mma<bf16_t>::mma(fb[ks][j], fa[ks][i], acc[i][j]);
                    }
                }
                st = st == NS - 1 ? 0 : st + 1;
            }
            wait_vmcnt_lgkm0<0>();
        } else {
            constexpr int CA = TA::PER_THREAD, CB = TB::PER_THREAD;
            uint32_t offA[CA], offB[CB], dstA[CA], dstB[CB];
            int kcA[CA], kcB[CB];
            auto geom = [&](auto tile, uint32_t& off, uint32_t& dst, int& kc, int i, int ld, int r0, int r_lim) {
                typedef decltype(tile) TT;
                const int q = threadIdx.x + i * SM::NT;
                const int row = q / TT::CPR, c = q % TT::CPR;
                dst = (uint32_t)((row * TT::CPR + (c ^ TT::swz(row))) * 16);
                if (TT::IS_KC) {
                    off = (uint32_t)((r0 + row) * ld + c * 8) * 4u;
                    kc = c * 8;
                } else {
                    off = r0 + c * 8 < r_lim ? (uint32_t)(row * ld + r0 + c * 8) * 4u : BUF_OOB;
                    kc = 0;
                }
            };
#pragma unroll
            for (int i = 0; i < CB; ++i) geom(TB(), offB[i], dstB[i], kcB[i], i, p.ldb, w.n0, p.N);
            const size_t rangeB = (size_t)(B_KC ? p.N : w.k_lim) * p.ldb * 4;
            auto load8 = [&](__amdgpu_buffer_rsrc_t rs, uint32_t off, u32x4_t (&r)[2]) {
                r[0] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
                r[1] = __builtin_amdgcn_raw_buffer_load_b128(rs, off == BUF_OOB ? BUF_OOB : off + 16, 0, 0);
            };
            // requests slab kt (zeros past the end) into a register set
            struct Slab { u32x4_t a[CA][2], b[CB][2]; };
            auto fetch_b = [&](int kt, Slab& r) {
                const int k0 = kt < nk ? kt * BK : 0;
                const size_t sh = (size_t)(B_KC ? k0 : k0 * p.ldb) * 4;
                const __amdgpu_buffer_rsrc_t rs = buf_rsrc((const char*)gB + sh, kt >= nk ? 0 : (B_KC ? rangeB : (rangeB > sh ? rangeB - sh : 0)));
#pragma unroll
                for (int i = 0; i < CB; ++i) load8(rs, (B_KC && KG && kcB[i] + k0 >= w.k_lim) ? BUF_OOB : offB[i], r.b[i]);
            };
            Slab s0, s1;
            fetch_b(0, s0);                  // B first: A is not touched before the rows in use are known
            fetch_b(1, s1);
            if (direct && !w.arrived(p)) continue;
            live = w.m0 + wm * (BM / 2) < w.m_lim;
#pragma unroll
            for (int i = 0; i < CA; ++i) geom(TA(), offA[i], dstA[i], kcA[i], i, p.lda, w.m0, w.m_lim);
            const size_t rangeA = (size_t)(A_KC ? w.m_lim : w.k_lim) * p.lda * 4;
            auto fetch_a = [&](int kt, Slab& r) {
                const int k0 = kt < nk ? kt * BK : 0;
                const size_t sh = (size_t)(A_KC ? k0 : k0 * p.lda) * 4;
                const __amdgpu_buffer_rsrc_t rs = buf_rsrc((const char*)gA + sh, kt >= nk ? 0 : (A_KC ? rangeA : (rangeA > sh ? rangeA - sh : 0)));
#pragma unroll
                for (int i = 0; i < CA; ++i) load8(rs, (A_KC && KG && kcA[i] + k0 >= w.k_lim) ? BUF_OOB : offA[i], r.a[i]);
            };
            auto put = [&](unsigned char* st, const Slab& r) {      // a fetched slab, split, into a stage
#pragma unroll
                for (int i = 0; i < CA; ++i) {
                    u32x4_t h, m, l;
                    split3_rne(r.a[i], h, m, l);
                    *reinterpret_cast<u32x4_t*>(st + dstA[i]) = h;
                    *reinterpret_cast<u32x4_t*>(st + TA::BYTES + dstA[i]) = m;
                    *reinterpret_cast<u32x4_t*>(st + 2 * TA::BYTES + dstA[i]) = l;
                }
#pragma unroll
                for (int i = 0; i < CB; ++i) {
                    u32x4_t h, m, l;
                    split3_rne(r.b[i], h, m, l);
                    unsigned char* d = st + 3 * TA::BYTES + dstB[i];
                    *reinterpret_cast<u32x4_t*>(d) = h;
                    *reinterpret_cast<u32x4_t*>(d + TB::BYTES) = m;
                    *reinterpret_cast<u32x4_t*>(d + 2 * TB::BYTES) = l;
                }
            };
            // One slab: its products, and under them the split of the next one (an MFMA occupies the matrix
            // pipe for 32 cycles, in which the wave issues up to six vector instructions for nothing).
            auto slab = [&](int kt, Slab& nxt, Slab& spare) {
                const unsigned char* st = smem_raw + (kt & 1) * SM::STAGE;
                fetch_a(kt + 2, spare);
                fetch_b(kt + 2, spare);
                bf16x8_t fa[KS][3][TM], fb[KS][3][TN];
// in the order in which the products below need them
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        constexpr int OA[3] = {2, 0, 1}, OB[3] = {0, 2, 1};
#pragma unroll
                        for (int i = 0; i < TM; ++i) fa[ks][OA[u]][i] = TA::frag(st + OA[u] * TA::BYTES, wm * (BM / 2) + i * 32, wk * KS + ks, lane);
#pragma unroll
                        for (int j = 0; j < TN; ++j) fb[ks][OB[u]][j] = TB::frag(st + 3 * TA::BYTES + OB[u] * TB::BYTES, wn * (BN / 2) + j * 32, wk * KS + ks, lane);
                    }
                put(smem_raw + ((kt + 1) & 1) * SM::STAGE, nxt);
                // smallest products first; mid*lo, lo*mid and lo*lo (below 2^-26 of the product) are left out
                constexpr int QA[6] = {2, 0, 1, 1, 0, 0}, QB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int q = 0; q < 6; ++q)
#pragma unroll
                        for (int i = 0; i < TM; ++i)
#pragma unroll
                            for (int j = 0; j < TN; ++j) acc[i][j] = Mma<bf16_t>::mma(fb[ks][QB[q]][j], fa[ks][QA[q]][i], acc[i][j]);
                constexpr int NRD = 3 * (TM * (A_KC ? 1 : 2) + TN * (B_KC ? 1 : 2)), NMF = 6 * TM * TN;
                constexpr int NV = (44 * (CA + CB) + KS * NMF - 1) / (KS * NMF);
                __builtin_amdgcn_sched_group_barrier(0x020, 2 * (CA + CB), 0);       // the loads of the slab after next
                __builtin_amdgcn_sched_group_barrier(0x100, NRD, 0);                 // fragments of the first k-step
#pragma unroll
                for (int m = 0; m < KS * NMF; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, NV, 0);
                    if (m < NMF * (KS - 1)) __builtin_amdgcn_sched_group_barrier(0x100, (NRD + NMF - 1) / NMF, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x200, 3 * (CA + CB), 0);
                __builtin_amdgcn_sched_barrier(0);
                // LDS writes of this wave are done and the workgroup meets; loads stay in flight
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            };
            fetch_a(0, s0);
            fetch_a(1, s1);
            put(smem_raw, s0);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            for (int kt = 0; kt < nk; kt += 2) {
                slab(kt, s1, s0);
                if (kt + 1 < nk) slab(kt + 1, s0, s1);
            }
        }
        __syncthreads();             // the strips lie over the ring
        if constexpr (KW > 1) {      // the groups' partial sums, added in group order
            float4* red = reinterpret_cast<float4*>(smem_raw);
            constexpr int PW = TM * TN * 4 * 64;     // float4 per wave
            if (wk > 0) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            red[(wave - 4) * PW + ((i * TN + j) * 4 + q) * 64 + lane] =
                                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
            }
            __syncthreads();
            if (wk == 0) {
#pragma unroll
                for (int k_ = 1; k_ < KW; ++k_)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const float4 x4 = red[(wave + 4 * (k_ - 1)) * PW + ((i * TN + j) * 4 + q) * 64 + lane];
                                acc[i][j][4 * q] += x4.x; acc[i][j][4 * q + 1] += x4.y;
                                acc[i][j][4 * q + 2] += x4.z; acc[i][j][4 * q + 3] += x4.w;
                            }
            }
            __syncthreads();
        }

        // ---- epilogue: lane holds row l32 of a 32x32 tile, columns 8q + 4g + 0..3 in registers 4q..4q+3
        constexpr int V = EPI == EPI_F32 ? 4 : 16 / (int)sizeof(T);      // elements per lane and store
        constexpr int WC = BN / 2, LPR = WC / V, RPI = 64 / LPR, NIT = 32 / RPI;
        constexpr uint32_t OSZ = EPI == EPI_F32 ? 4u : (uint32_t)sizeof(T);
        if (live && wk == 0) {
            if constexpr (SPLIT) {
                if (__builtin_expect(split_in_doubt<TM, TN>(acc, w.m_lim - w.m0 - wm * (BM / 2), l32), 0))
                    redo_f32<A_KC, B_KC, TM, TN>(acc, more < 0 ? 1 : 0, w.e, w.m0 + wm * (BM / 2), w.m_lim, w.n0 + wn * (BN / 2), l32, g);
            }
            float* strip = reinterpret_cast<float*>(smem_raw) + wave * 32 * SM::STRIP_LD;
            const int er = lane / LPR, ec = (lane - er * LPR) * V;
            const int ncol = w.n0 + wn * WC + ec;
            const bool col_ok = ncol < p.N;
            const size_t obase = (size_t)w.e * p.strideO, obytes = (size_t)w.m_lim * p.ldo * OSZ;
            const __amdgpu_buffer_rsrc_t o0 = buf_rsrc((const char*)p.out0 + obase * OSZ, obytes);
            const __amdgpu_buffer_rsrc_t o1 = buf_rsrc(EPI == EPI_H_DACT ? (const char*)p.out1 + obase * OSZ : nullptr, EPI == EPI_H_DACT ? obytes : 0);
            const __amdgpu_buffer_rsrc_t ax = buf_rsrc(EPI == EPI_MUL ? (const char*)p.aux + obase * OSZ : nullptr, EPI == EPI_MUL ? obytes : 0);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int mb = w.m0 + wm * (BM / 2) + i * 32;
                if (mb >= w.m_lim) break;
                auto out_off = [&](int it) { return col_ok ? (uint32_t)(((size_t)(mb + er + it * RPI) * p.ldo + ncol) * OSZ) : BUF_OOB; };
                float aux[EPI == EPI_MUL ? NIT : 1][V];
                if constexpr (EPI == EPI_MUL) {
#pragma unroll
                    for (int it = 0; it < NIT; ++it) BufChunk<T>::load(ax, out_off(it), aux[it]);
                }
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<float4*>(strip + l32 * SM::STRIP_LD + j * 32 + 8 * q + 4 * g) =
                            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                auto vec = [&](int it) {
                    float v[V];
#pragma unroll
                    for (int c = 0; c < V / 4; ++c) {
                        const float4 x4 = *reinterpret_cast<const float4*>(strip + (er + it * RPI) * SM::STRIP_LD + ec + 4 * c);
                        v[4 * c] = x4.x; v[4 * c + 1] = x4.y; v[4 * c + 2] = x4.z; v[4 * c + 3] = x4.w;
                    }
                    const uint32_t off = out_off(it);
                    if constexpr (EPI == EPI_F32) {
                        BufChunk<float>::store(o0, off, v);
                    } else if constexpr (EPI == EPI_STORE) {
                        BufChunk<T>::store(o0, off, v);
                    } else if constexpr (EPI == EPI_MUL) {
#pragma unroll
                        for (int c = 0; c < V; ++c) v[c] *= aux[it][c];
                        BufChunk<T>::store(o0, off, v);
                    } else {
                        float a[V], h[V];
#pragma unroll
                        for (int c = 0; c < V; ++c) act_both<sizeof(T) == 2, ACT>(v[c], h[c], a[c]);
                        if constexpr (EPI == EPI_H_DACT) {
                            if (p.drop_thr) {
#pragma unroll
                                for (int c4 = 0; c4 < V / 4; ++c4) {
                                    uint32_t nw[4];
                                    noise_words(obase + (size_t)(mb + er + it * RPI) * p.ldo + ncol + 4 * c4, MOE_STREAM_DROPOUT, p.seed, nw);
#pragma unroll
                                    for (int c = 0; c < 4; ++c) {
                                        const float sc = nw[c] >= p.drop_thr ? p.drop_scale : 0.0f;
                                        h[4 * c4 + c] *= sc;
                                        a[4 * c4 + c] *= sc;
                                    }
                                }
                            }
                            BufChunk<T>::store(o0, off, a);
                            BufChunk<T>::store(o1, off, h);
                        } else {
                            BufChunk<T>::store(o0, off, h);
                        }
                    }
                };
                if constexpr (EPI == EPI_H_DACT || EPI == EPI_H) {
#pragma unroll 1
                    for (int it = 0; it < NIT; ++it) vec(it);
                } else {
#pragma unroll
                    for (int it = 0; it < NIT; ++it) vec(it);
                }
            }
        }
        __syncthreads();             // the next tile's slabs overwrite the strips
    }
    return w.where();
}

template <typename T, int BM, int BN, int KW, int NS, bool A_KC, bool B_KC, int EPI, int ACT, bool KG>
__global__ __launch_bounds__(256 * KW, (KW * MidSmem<T, BM, BN, KW, NS, A_KC, B_KC>::OCC)) void mid_gemm_kernel(const GemmArgs p) {
    mid_body<T, BM, BN, KW, NS, A_KC, B_KC, EPI, ACT, KG>(p, 0, {0, 0});
}
template <typename T, int BM, int BN, int KW, int NS, bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2, bool KG>
__global__ __launch_bounds__(256 * KW, (KW * MidSmem<T, BM, BN, KW, NS, A1, B1>::OCC)) void mid_gemm_pair_kernel(const GemmArgs p1, const GemmArgs p2) {
    const typename TileWalk<BM, BN>::Where w = mid_body<T, BM, BN, KW, NS, A1, B1, EPI1, 0, KG>(p1, p2.E * p2.tiles_m * p2.tiles_n, {0, 0});
    __syncthreads();      // every wave is done with the tile table of the first product
    mid_body<T, BM, BN, KW, NS, A2, B2, EPI2, 0, KG>(p2, -1, w);
}

// ---------------------------------------------------------------------------
// The smallest fp32 products: 32 x 32 tiles, one per workgroup of four waves, which take the reduction's 32-deep
// chunks in turn.  What bounds these launches is latency, not work: with 64 x 64 tiles, slabs staged through LDS and a
// table of tiles, h W2 with 256 rows, d = 64, f = 256 took 8.2 us, of which 1.8 went to the table and 0.9 to each of its
// four slabs (LDS traffic of the split planes and a barrier).  Here a wave's fragments come straight from memory into
// registers, two chunks ahead, and are split there; nothing is shared before the four partial sums meet in LDS, and
// each wave finishes a quarter of the columns.  Every operand element is split by each tile that needs it, so this is
// for products whose tiles would leave much of the chip idle.  The four launches of 256 tokens, d = 64, f = 256,
// 4 experts: 7.0, 8.1, 7.7, 9.5 -> 4.8, 5.2, 4.6, 5.8 us; of 777 tokens, d = 136, f = 328, 5 experts, top-2:
// 12.4, 11.1, 14.3, 12.9 -> 7.4, 6.4, 12.6, 9.0.  Three waves per SIMD: four of the seven instances then spill 2 - 4
// registers (12 - 20 bytes a lane) outside of the loop over chunks; with four waves (128 registers) 10 - 24 spill.
// ---------------------------------------------------------------------------
enum { THIN = 32, THIN_WAVES = 4, THIN_OCC = 3, THIN_GRID = 8 };      // waves per SIMD = workgroups that a CU holds; most of a launch per CU

template <bool A_KC, bool B_KC, int EPI, int ACT>
__device__ __forceinline__ typename TileWalk<THIN, THIN>::Where thin_body(const GemmArgs& p, int more, typename TileWalk<THIN, THIN>::Where before) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    constexpr int SUMS = THIN_WAVES * THIN * THIN * 4;
    float4* red = reinterpret_cast<float4*>(smem_raw);
    TileWalk<THIN, THIN> w;
    const bool direct = p.direct_count > 0;
    if (direct) {
        if (!w.only(p)) return w.where();
    } else if (p.E <= MOE_WAVE) {
        w.count(p);
        w.begin(p, more < 0 ? before.total : more, more < 0);
    } else {
        TileWalk<THIN, THIN>::build(p, smem_raw + SUMS);
        if (more < 0) w.resume(p, before, smem_raw + SUMS); else w.start(p, smem_raw + SUMS, more);
    }
    for (bool more_tiles = direct || w.next(p); more_tiles; more_tiles = !direct && w.next(p)) {
        const int nc = (w.k_lim + 31) >> 5;
        // A chunk's element (r, k0 + 16g + 8s + j) is entry j of k-step s: the order of a reduction is free, and so a
        // lane of a k-contiguous operand reads 64 consecutive bytes and its two lanes a whole line.
        struct Chunk { u32x4_t q[4]; };
        const __amdgpu_buffer_rsrc_t rsB = buf_rsrc((const float*)p.B + (size_t)w.e * p.strideB, (size_t)(B_KC ? p.N : w.k_lim) * p.ldb * 4);
        const int rA = w.m0 + l32, rB = w.n0 + l32;
        auto load = [&](auto kc, __amdgpu_buffer_rsrc_t rs, int r, int r_lim, int ld, int c) {
            Chunk v;
            const int k = 32 * c + 16 * g;
            if constexpr (decltype(kc)::value) {
                const uint32_t off = (uint32_t)(r * ld + k) * 4u;        // rows >= r_lim lie beyond the range
#pragma unroll
                for (int i = 0; i < 4; ++i) v.q[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, k + 4 * i < w.k_lim ? off + 16 * i : BUF_OOB, 0, 0);
            } else {
                const uint32_t off = r < r_lim ? (uint32_t)(k * ld + r) * 4u : BUF_OOB;     // k >= k_lim lies beyond it
#pragma unroll
                for (int i = 0; i < 16; ++i) v.q[i >> 2][i & 3] = __builtin_amdgcn_raw_buffer_load_b32(rs, off + (uint32_t)(i * ld) * 4u, 0, 0);
            }
            return v;
        };
        struct Both { Chunk a, b; };
        auto load_b = [&](int c) { return load(std::integral_constant<bool, B_KC>(), rsB, rB, p.N, p.ldb, c); };
        // The products of the leading parts are summed apart from the five corrections (2^-8 of them and less): one
        // rounding at the size of the sum per 16 products instead of six, and two chains of MFMAs instead of one.
        f32x16_t acc, fine;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = fine[v] = 0.0f;
        auto multiply = [&](const Both& v) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const u32x4_t wa[2] = {v.a.q[2 * s], v.a.q[2 * s + 1]}, wb[2] = {v.b.q[2 * s], v.b.q[2 * s + 1]};
                u32x4_t fa[3], fb[3];
                split3_rne(wa, fa[0], fa[1], fa[2]);
                split3_rne(wb, fb[0], fb[1], fb[2]);
                auto mma = [&](int qa, int qb, f32x16_t c) { return Mma<bf16_t>::mma(__builtin_bit_cast(bf16x8_t, fb[qb]), __builtin_bit_cast(bf16x8_t, fa[qa]), c); };
                acc = mma(0, 0, acc);
                constexpr int QA[5] = {2, 0, 1, 1, 0}, QB[5] = {0, 2, 1, 0, 1};    // smallest products first
#pragma unroll
                for (int q = 0; q < 5; ++q) fine = mma(QA[q], QB[q], fine);
            }
        };
        // issued in this order and not rearranged: the waits in the loop count on it.  B first: A is not touched before the
        // rows in use are known.
        Both v0, v1;
        v0.b = load_b(wave);
        __builtin_amdgcn_sched_barrier(0);
        v1.b = load_b(wave + THIN_WAVES);
        __builtin_amdgcn_sched_barrier(0);
        if (direct && !w.arrived(p)) continue;
        const __amdgpu_buffer_rsrc_t rsA = buf_rsrc((const float*)p.A + (size_t)w.e * p.strideA, (size_t)(A_KC ? w.m_lim : w.k_lim) * p.lda * 4);
        auto load_a = [&](int c) { return load(std::integral_constant<bool, A_KC>(), rsA, rA, w.m_lim, p.lda, c); };
        auto fetch = [&](int c) {
            Both v;
            v.b = load_b(c);
            v.a = load_a(c);
            return v;
        };
        v0.a = load_a(wave);
        __builtin_amdgcn_sched_barrier(0);
        v1.a = load_a(wave + THIN_WAVES);
        __builtin_amdgcn_sched_barrier(0);
        // this wave's share of the result: row l32, columns 8 wave + 4g + 0..3 of the tile
        const int row = w.m0 + l32, col = w.n0 + 8 * wave + 4 * g;
        const uint32_t off = col < p.N ? (uint32_t)((size_t)row * p.ldo + col) * 4u : BUF_OOB;
        const size_t obase = (size_t)w.e * p.strideO;
        const size_t obytes = (size_t)w.m_lim * p.ldo * 4;       // the expert's rows in use
        float aux[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (EPI == EPI_MUL) BufChunk<float>::load(buf_rsrc((const float*)p.aux + obase, obytes), off, aux);
        for (int c = wave; c < nc; c += 2 * THIN_WAVES) {
            multiply(v0);
            __builtin_amdgcn_sched_barrier(0);
            v0 = fetch(c + 2 * THIN_WAVES);
            __builtin_amdgcn_sched_barrier(0);
            if (c + THIN_WAVES >= nc) break;
            multiply(v1);
            __builtin_amdgcn_sched_barrier(0);
            v1 = fetch(c + 3 * THIN_WAVES);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] += fine[v];
#pragma unroll
        for (int q = 0; q < 4; ++q) red[(wave * 4 + q) * 64 + lane] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        __syncthreads();
        f32x16_t sum[1][1];
#pragma unroll
        for (int v = 4; v < 16; ++v) sum[0][0][v] = 0.0f;
        static_assert(THIN_WAVES == 4, "the sum below");
        float4 part[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) part[i] = red[(i * 4 + wave) * 64 + lane];
        sum[0][0][0] = (part[0].x + part[1].x) + (part[2].x + part[3].x);
        sum[0][0][1] = (part[0].y + part[1].y) + (part[2].y + part[3].y);
        sum[0][0][2] = (part[0].z + part[1].z) + (part[2].z + part[3].z);
        sum[0][0][3] = (part[0].w + part[1].w) + (part[2].w + part[3].w);
        if (!direct) __syncthreads();      // the next tile's sums go to the same place
        float z[4] = {sum[0][0][0], sum[0][0][1], sum[0][0][2], sum[0][0][3]};
        if (__builtin_expect(split_in_doubt<1, 1>(sum, w.m_lim - w.m0, l32), 0)) {
            redo_f32<A_KC, B_KC, 1, 1>(sum, more < 0 ? 1 : 0, w.e, w.m0, w.m_lim, w.n0, l32, g);
#pragma unroll
            for (int r = 0; r < 4; ++r) z[r] = wave == 0 ? sum[0][0][r] : wave == 1 ? sum[0][0][4 + r] : wave == 2 ? sum[0][0][8 + r] : sum[0][0][12 + r];
        }
        const __amdgpu_buffer_rsrc_t o0 = buf_rsrc((const float*)p.out0 + obase, obytes);
        if constexpr (EPI == EPI_H_DACT || EPI == EPI_H) {
            float h[4], a[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) act_both<false, ACT>(z[r], h[r], a[r]);
            if constexpr (EPI == EPI_H_DACT) {
                if (p.drop_thr) {
                    uint32_t nw[4];
                    noise_words(obase + (size_t)row * p.ldo + col, MOE_STREAM_DROPOUT, p.seed, nw);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float sc = nw[r] >= p.drop_thr ? p.drop_scale : 0.0f;
                        h[r] *= sc;
                        a[r] *= sc;
                    }
                }
                BufChunk<float>::store(o0, off, a);
                BufChunk<float>::store(buf_rsrc((const float*)p.out1 + obase, obytes), off, h);
            } else {
                BufChunk<float>::store(o0, off, h);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) z[r] = EPI == EPI_MUL ? z[r] * aux[r] : z[r];
            BufChunk<float>::store(o0, off, z);
        }
    }
    return w.where();
}

template <bool A_KC, bool B_KC, int EPI, int ACT>
__global__ __launch_bounds__(64 * THIN_WAVES, THIN_OCC) void thin_gemm_kernel(const GemmArgs p) {
    thin_body<A_KC, B_KC, EPI, ACT>(p, 0, {0, 0});
}
template <bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2>
__global__ __launch_bounds__(64 * THIN_WAVES, THIN_OCC) void thin_gemm_pair_kernel(const GemmArgs p1, const GemmArgs p2) {
    const typename TileWalk<THIN, THIN>::Where w = thin_body<A1, B1, EPI1, 0>(p1, p2.E * p2.tiles_m * p2.tiles_n, {0, 0});
    __syncthreads();      // every wave is done with the sums and the tile table of the first product
    thin_body<A2, B2, EPI2, 0>(p2, -1, w);
}

// Number of compute units of the current device (looked up once per device).
static int num_cus() {
    static int cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
    if (n == 0) {
        int v = 0;
        n = (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ? v : 256;
        __atomic_store_n(&cached[dev], n, __ATOMIC_RELAXED);
    }
    return n;
}

// one persistent workgroup per CU (its LDS footprint allows no second one), in groups of 8 so
// that every XCD gets the same number; never more than there could be tiles
static int gemm_grid(long long tiles) {
    const long long most = (tiles + 7) / 8;
    int per_xcd = num_cus() / 8;
    if (per_xcd < 1) per_xcd = 1;
    if (per_xcd > most) per_xcd = (int)most;
    return per_xcd * 8;
}

static void set_tiles(GemmArgs& p, int BM, int BN, int E) {
    p.tiles_m = ceil_div(p.M, BM);
    p.tiles_n = ceil_div(p.N, BN);
    p.E = E;
}
static long long all_tiles(const GemmArgs& p) { return (long long)p.E * p.tiles_m * p.tiles_n; }

// smaller tiles: `occ` workgroups per CU.  Of a launch of two products (p2, or null) each has its own eighths of an XCD, as
// TileWalk::begin() counts them: with one workgroup too few for that the first product's tiles, or the last of the second's,
// are all one XCD's (fp32, 19 experts of 55 rows, d = 96, f = 384, dxd with dW1, 798 tiles: 800 workgroups 17.2 us, 808 8.2).
static int mid_grid(const GemmArgs& p, const GemmArgs* p2, int occ) {
    const long long most = (all_tiles(p) + 7) / 8 + (p2 ? (all_tiles(*p2) + 7) / 8 : 0);
    long long per_xcd = (long long)num_cus() / 8 * occ;
    if (per_xcd < 1) per_xcd = 1;
    if (per_xcd > most) per_xcd = most;
    return (int)per_xcd * 8;
}

// One tile per workgroup, addressed without the experts' row counts, where at least four of five of all tiles that there
// could be are expected to hold rows and each has a CU to itself: an expert's tiles are an XCD's, and with a skewed gate the
// ones in use would share some of the CUs while the others' idle.  Expert FFN forward, addressed so against walked by the
// counts, Zipf gate: 8 experts of 117 slots, 304 tiles, 24 us and 19; all tokens on one of 5 experts, 1320 tiles of 32 x 32,
// h W2 44 us and 30; a fifth of the slots empty, 302 tiles, 16.5 and 12.4.  One expert's rows are known: with none of its
// tiles empty, as many as the launch may have workgroups (`occ` per CU).  p2: the launch's second product or null.  Returns the workgroups per
// XCD, 0 where the tiles are walked instead.
static int set_direct(GemmArgs& p, GemmArgs* p2, int rows, int side, int occ) {
    const long long s1 = (all_tiles(p) + 7) / 8, s2 = p2 ? (all_tiles(*p2) + 7) / 8 : 0;
    const int filled = ceil_div(rows, side), per_cu = p.E == 1 && p.tiles_m == filled ? occ : 1;
    if (4 * p.tiles_m > 5 * filled || s1 + s2 > (long long)num_cus() / 8 * per_cu) return 0;
    for (GemmArgs* q : {&p, p2}) {
        if (!q) continue;
        const int per_e = q->tiles_m * q->tiles_n;
        q->direct_first = q == &p ? 0 : (int)s1;
        q->direct_count = (int)all_tiles(*q);
        q->inv_expert = per_e > 1 ? (uint32_t)((1ull << 32) / per_e + 1) : 0;       // exact for t d < 2^32; 0: d = 1
        q->inv_m = q->tiles_m > 1 ? (uint32_t)((1ull << 32) / q->tiles_m + 1) : 0;
    }
    return (int)(s1 + s2);
}

template <typename T, int BM, int BN, int KW, int NS, bool A_KC, bool B_KC, int EPI, int ACT>
static bool launch_mid(GemmArgs p, int rows, int E, hipStream_t st) {
    typedef MidSmem<T, BM, BN, KW, NS, A_KC, B_KC> SM;
    set_tiles(p, BM, BN, E);
    const int direct = set_direct(p, nullptr, rows, BM, SM::OCC);
    const size_t smem = SM::BYTES + WALK_BYTES;
    // a k-contiguous operand whose reduction length is not a multiple of the slab needs the guarded instance
    const bool kg = (A_KC || B_KC) && !p.var_k && p.K % SM::BK != 0;
    static unsigned long long opted[2] = {0, 0};
    auto kern = kg ? mid_gemm_kernel<T, BM, BN, KW, NS, A_KC, B_KC, EPI, ACT, true> : mid_gemm_kernel<T, BM, BN, KW, NS, A_KC, B_KC, EPI, ACT, false>;
    if (!lds_opt_in((const void*)kern, smem, &opted[kg])) return false;
    kern<<<direct ? 8 * direct : mid_grid(p, nullptr, SM::OCC), SM::NT, smem, st>>>(p);
    return true;
}

template <typename T, int BM, int BN, int KW, int NS, bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2>
static bool launch_mid_pair(GemmArgs p1, GemmArgs p2, int rows, int E, hipStream_t st) {
    typedef MidSmem<T, BM, BN, KW, NS, A1, B1> SM;
    set_tiles(p1, BM, BN, E);
    set_tiles(p2, BM, BN, E);
    const int direct = set_direct(p1, &p2, rows, BM, SM::OCC);
    const size_t smem = SM::BYTES + WALK_BYTES;
    const bool kg = ((A1 || B1) && !p1.var_k && p1.K % SM::BK != 0) || ((A2 || B2) && !p2.var_k && p2.K % SM::BK != 0);
    static unsigned long long opted[2] = {0, 0};
    auto kern = kg ? mid_gemm_pair_kernel<T, BM, BN, KW, NS, A1, B1, EPI1, A2, B2, EPI2, true> : mid_gemm_pair_kernel<T, BM, BN, KW, NS, A1, B1, EPI1, A2, B2, EPI2, false>;
    if (!lds_opt_in((const void*)kern, smem, &opted[kg])) return false;
    kern<<<direct ? 8 * direct : mid_grid(p1, &p2, SM::OCC), SM::NT, smem, st>>>(p1, p2);
    return true;
}

template <bool A_KC, bool B_KC, int EPI, int ACT>
static bool launch_thin(GemmArgs p, int rows, int E, hipStream_t st) {
    set_tiles(p, THIN, THIN, E);
    const int direct = set_direct(p, nullptr, rows, THIN, THIN_GRID);
    const size_t smem = THIN_WAVES * THIN * THIN * 4 + WALK_BYTES;
    thin_gemm_kernel<A_KC, B_KC, EPI, ACT><<<direct ? 8 * direct : mid_grid(p, nullptr, THIN_GRID), 64 * THIN_WAVES, smem, st>>>(p);
    return true;
}

template <bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2>
static bool launch_thin_pair(GemmArgs p1, GemmArgs p2, int rows, int E, hipStream_t st) {
    set_tiles(p1, THIN, THIN, E);
    set_tiles(p2, THIN, THIN, E);
    const int direct = set_direct(p1, &p2, rows, THIN, THIN_GRID);
    const size_t smem = THIN_WAVES * THIN * THIN * 4 + WALK_BYTES;
    thin_gemm_pair_kernel<A1, B1, EPI1, A2, B2, EPI2><<<direct ? 8 * direct : mid_grid(p1, &p2, THIN_GRID), 64 * THIN_WAVES, smem, st>>>(p1, p2);
    return true;
}

template <bool A_KC, bool B_KC, int EPI, int ACT>
static bool launch_big(GemmArgs p, int E, hipStream_t st) {
    typedef GemmSmem<BIG_M, BIG_N, BIG_K, A_KC, B_KC, BIG_WN> SM;
    set_tiles(p, BIG_M, BIG_N, E);
    const size_t smem = SM::BYTES + WALK_BYTES;
    const bool kg = (A_KC || B_KC) && !p.var_k && p.K % BIG_K != 0;
    static unsigned long long opted[2] = {0, 0};
    auto kern = kg ? grouped_gemm_kernel<BIG_M, BIG_N, BIG_K, A_KC, B_KC, EPI, ACT, BIG_WN, true>
                   : grouped_gemm_kernel<BIG_M, BIG_N, BIG_K, A_KC, B_KC, EPI, ACT, BIG_WN, false>;
    if (!lds_opt_in((const void*)kern, smem, &opted[kg])) return false;
    kern<<<gemm_grid(all_tiles(p)), SM::NT, smem, st>>>(p);
    return true;
}

template <bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2>
static bool launch_big_pair(GemmArgs p1, GemmArgs p2, int E, hipStream_t st) {
    typedef GemmSmem<BIG_M, BIG_N, BIG_K, A1, B1, BIG_WN> SM1;
    typedef GemmSmem<BIG_M, BIG_N, BIG_K, A2, B2, BIG_WN> SM2;
    static_assert(SM1::NT == SM2::NT, "one workgroup shape");
    set_tiles(p1, BIG_M, BIG_N, E);
    set_tiles(p2, BIG_M, BIG_N, E);
    const size_t smem = (SM1::BYTES > SM2::BYTES ? SM1::BYTES : SM2::BYTES) + WALK_BYTES;
    const bool kg = ((A1 || B1) && !p1.var_k && p1.K % BIG_K != 0) || ((A2 || B2) && !p2.var_k && p2.K % BIG_K != 0);
    static unsigned long long opted[2] = {0, 0};
    auto kern = kg ? grouped_gemm_pair_kernel<BIG_M, BIG_N, BIG_K, A1, B1, EPI1, A2, B2, EPI2, BIG_WN, true>
                   : grouped_gemm_pair_kernel<BIG_M, BIG_N, BIG_K, A1, B1, EPI1, A2, B2, EPI2, BIG_WN, false>;
    if (!lds_opt_in((const void*)kern, smem, &opted[kg])) return false;
    kern<<<gemm_grid(all_tiles(p1) + all_tiles(p2)), SM1::NT, smem, st>>>(p1, p2);
    return true;
}

// ---- which tile ------------------------------------------------------------------
// The expert counts are on the device; the host knows the mean demand T k / E and the capacity and takes the smaller
// of the two for the rows of every expert.  With a skewed gate that is more than the mean of what experts hold: those
// above the capacity drop rows and the others have fewer.  (Six experts, T = 5003, top-2, Zipf gate: 1668 against 1392 on
// average, so that h W2 with d = 776, f = 3080 gets the large tile where the small one measured faster.)
enum FfnTile { TILE_32, TILE_64, TILE_128_PAIRED, TILE_128, TILE_256 };      // PAIRED: two wave groups share a tile
// Tiles of a given side of one product: `rows` output rows (the expert's, or all M of a weight gradient), N columns.
static double tiles_expected(int rows, int N, int side, int E) { return (double)E * ceil_div(rows, side) * ceil_div(N, side); }
// bf16, experts with more than 128 rows: time goes with the number of whole rounds.  The 256 x 256
// kernel runs one tile per CU and round; the 128 x 128 one runs two per CU, each a quarter of the
// work at 0.78 of the rate (0.74 - 0.87 over the six products at 32 experts of 1024 rows, d = 1024,
// f = 4096).  h W2 with six experts of 1440 rows, d = 776, f = 3080 (144 large tiles, 504 small ones):
// 65 us against 80; with 16 experts of 1024 rows, d = 768, f = 3072 (192 and 768): 118 against 90.
static bool prefer_mid(double t256, double t128) {
    const double cus = num_cus();
    return ceil(t128 / (2 * cus)) * (cus / 2) / 0.78 < ceil(t256 / cus) * cus;
}

// fp32, few tiles: 32 x 32 or 64 x 64, by the time (us) that each would take.  n32 and n64 tiles with reductions of k
// entries, and of the launch's second product m32 and m64 with reductions of l (none: 0).  After its start a launch lasts as
// long as its longest reduction (64 x 64: 0.016 us per entry; 32 x 32, where four waves share it: 0.0093) or as the most
// tiles that a CU gets (2.8 + 0.0135 per entry; 1.5 + 0.0048).  Fitted, as the factor on the estimate for 64 x 64 and the
// limit of 5.5 tiles per CU are, to 885 launches of 8 - 2500 rows, d = 32 - 1500, 1 - 64 experts, balanced and skewed: the form
// chosen is 2 % (one product) and 4 % (two) slower than the better one on average, where 64 x 64 alone would be 20 % slower.
// In us, 64 x 64 against 32 x 32, one product: 28 and 8 tiles 7 and 8 against 5 and 5 (256 tokens, d = 64); 150 and 550
// tiles 9.2 and 7.8 (777 tokens, d = 136); 264 and 990 of K = 176, two rounds against four, 14.9 and 12.0; 240 and 960 of
// K = 192, one round, 6.8 and 10.6; 504 and 1476 of K = 3864 138 and 159.  Two: 174 and 672 tiles, reductions of 1675
// rows, 33.6 and 17.5; 304 and 1200, of 2137, 44 and 28; 256 and 992, of 512 and 461, 12.3 and 17.4; 525 and 1845 21 and 62.
static FfnTile few_tiles(double n32, double n64, int k, double m32, double m64, int l) {
    const double cus = num_cus(), longest = k > l ? k : l;
    auto us = [&](double n, double m, double start, double chain, double tile, double entry) {
        return start + fmax(chain * longest, ceil((n + m) / cus) * (tile + entry * (n * k + m * l) / (n + m)));
    };
    const double us32 = us(n32, m32, 0.6, 0.0093, 1.5, 0.0048), us64 = us(n64, m64, 2.8, 0.016, 2.8, 0.0135);
    return n32 + m32 <= 5.5 * cus && us32 <= (m32 > 0.0 ? 1.25 : 1.15) * us64 ? TILE_32 : TILE_64;
}

// fp32: 64 x 64 tiles as long as 128 x 128 ones would leave much of the chip idle (five experts of 280
// rows, d = 136, f = 328: 10 us per product against 17 - 23); 128 x 128 with two wave groups that
// share a tile's slabs while there are few tiles per CU (248 tiles, f = 2048: 89 us against 124 with
// one group), with one group otherwise (992 tiles, d = 512: 105 against 117).
// Where 64 x 64 tiles it is, few_tiles() says whether they are computed as 32 x 32 ones.
// bf16: the same order.  64 x 64 (8 experts of 64 rows, d = 512, f = 2048: 7 and 11 us against 10 and
// 22 with 128 x 128, 17 and 39 with 256 x 256); with few rows per expert the weights' stream is the
// bound and two 128 x 128 workgroups per CU keep more of it in flight than one large one (107 experts
// of 7 rows, d = 1024, f = 4096: 169 us = 5.3 TB/s against 203).
static FfnTile tile_for(bool f32, int rows, int N, int K, int E) {
    const double cus = num_cus(), t128 = tiles_expected(rows, N, 128, E);
    if (f32 && t128 <= 0.6 * cus)
        return few_tiles(tiles_expected(rows, N, THIN, E), tiles_expected(rows, N, 64, E), K, 0, 0, 0);
    if (f32) return t128 <= 1.5 * cus ? TILE_128_PAIRED : TILE_128;
    if (t128 <= (rows <= 128 ? 1.0 : 0.5) * cus) return TILE_64;
    return rows <= 128 || prefer_mid(tiles_expected(rows, N, 256, E), t128) ? TILE_128 : TILE_256;
}

// Two products, `rows` rows by N1 columns and a weight gradient of M2 by N2: the same lines at higher tile
// counts, because the tiles of both are in the launch (fp32, 248 + 512 tiles: 185 us with two wave groups, 250 with
// one; 992 + 512: 197 and 179.  bf16, 8 experts of 64 rows, 32 + 512 tiles: 26 us with 64 x 64, 30 with 128 x 128, 41
// with 256 x 256).  The first product's reduction is N2 long, the second's `rows`.
// bf16, experts of at most 128 rows: half of a large tile is padding.  dz with dW2 (`first`) takes 128 x 128 (36 experts of
// 66 rows, d = 864, f = 2256: 90 us against 127 with 256 x 256; 81 of 11, d = 1064, f = 3368: 365 against 420; 24 of 74,
// d = 1200, f = 600: 25 against 49).  dxd with dW1, where one of the two products' reductions is long, takes it for up to ten
// tiles per CU (4 of 101, d = 968, f = 3840, 3.9 per CU: 42 against 70; 12 of 17, d = 1376, f = 2056, 9.3: 70 against 79);
// beyond, the rounds decide as with more rows (36 of 41, d = 1152, f = 4024, 42 per CU: 276 against 252; 64 of 46,
// d = f = 1512, 36: 235 against 206; 100 of 66, d = 560, f = 1776, 29: 150 against 202).
static FfnTile tile_for_pair(bool f32, bool first, int rows, int N1, int M2, int N2, int E) {
    const double cus = num_cus(), t128 = tiles_expected(rows, N1, 128, E) + tiles_expected(M2, N2, 128, E);
    if (f32 && t128 <= 0.75 * cus)
        return few_tiles(tiles_expected(rows, N1, THIN, E), tiles_expected(rows, N1, 64, E), N2, tiles_expected(M2, N2, THIN, E),
                         tiles_expected(M2, N2, 64, E), rows);
    if (f32) return t128 <= 4.0 * cus ? TILE_128_PAIRED : TILE_128;
    if (t128 <= (rows <= 128 ? 3.0 : 1.0) * cus) return TILE_64;
    if (rows <= 128 && (first || t128 <= 10.0 * cus)) return TILE_128;
    return prefer_mid(tiles_expected(rows, N1, 256, E) + tiles_expected(M2, N2, 256, E), t128) ? TILE_128 : TILE_256;
}

template <typename T, bool A_KC, bool B_KC, int EPI, int ACT = 0>
static bool launch_gemm(const GemmArgs& p, int rows, int E, hipStream_t st) {
    const FfnTile t = tile_for(sizeof(T) == 4, rows, p.N, p.K, E);
    if constexpr (sizeof(T) == 4) {
        if (t == TILE_32) return launch_thin<A_KC, B_KC, EPI, ACT>(p, rows, E, st);
        if (t == TILE_64) return launch_mid<T, 64, 64, 2, 2, A_KC, B_KC, EPI, ACT>(p, rows, E, st);
        if (t == TILE_128_PAIRED) return launch_mid<T, 128, 128, 2, 2, A_KC, B_KC, EPI, ACT>(p, rows, E, st);
        return launch_mid<T, 128, 128, 1, 2, A_KC, B_KC, EPI, ACT>(p, rows, E, st);
    } else {
        if (t == TILE_64) return launch_mid<T, 64, 64, 1, 3, A_KC, B_KC, EPI, ACT>(p, rows, E, st);
        if (t == TILE_128) return launch_mid<T, 128, 128, 1, 2, A_KC, B_KC, EPI, ACT>(p, rows, E, st);
        return launch_big<A_KC, B_KC, EPI, ACT>(p, E, st);
    }
}

template <typename T, bool A1, bool B1, int EPI1, bool A2, bool B2, int EPI2>
static bool launch_gemm_pair(const GemmArgs& p1, const GemmArgs& p2, int rows, int E, hipStream_t st) {
    const FfnTile t = tile_for_pair(sizeof(T) == 4, EPI1 == EPI_MUL, rows, p1.N, p2.M, p2.N, E);
    if constexpr (sizeof(T) == 4) {
        if (t == TILE_32) return launch_thin_pair<A1, B1, EPI1, A2, B2, EPI2>(p1, p2, rows, E, st);
        if (t == TILE_64) return launch_mid_pair<T, 64, 64, 2, 2, A1, B1, EPI1, A2, B2, EPI2>(p1, p2, rows, E, st);
        if (t == TILE_128_PAIRED) return launch_mid_pair<T, 128, 128, 2, 2, A1, B1, EPI1, A2, B2, EPI2>(p1, p2, rows, E, st);
        return launch_mid_pair<T, 128, 128, 1, 2, A1, B1, EPI1, A2, B2, EPI2>(p1, p2, rows, E, st);
    } else {
        if (t == TILE_64) return launch_mid_pair<T, 64, 64, 1, 3, A1, B1, EPI1, A2, B2, EPI2>(p1, p2, rows, E, st);
        if (t == TILE_128) return launch_mid_pair<T, 128, 128, 1, 2, A1, B1, EPI1, A2, B2, EPI2>(p1, p2, rows, E, st);
        return launch_big_pair<A1, B1, EPI1, A2, B2, EPI2>(p1, p2, E, st);
    }
}

size_t ffn_bwd_ws_bytes(const moe_shape* s) {
    return align_up((size_t)s->E * s->capacity * s->d_ff * elem_bytes(s->dtype), 256);
}

// Per-expert operand slices are addressed with 32-bit byte offsets.
static int check_slice_limits(const moe_shape* s) {
    const long long big = (long long)(s->d_model > s->d_ff ? s->d_model : s->d_ff);
    if (((long long)s->capacity + 512) * big * 4 >= (1ll << 31) || (long long)s->d_model * s->d_ff * 4 >= (1ll << 31))
        return MOE_ERR_SHAPE;
    return MOE_OK;
}

static int expected_rows(const moe_shape* s) {
    const int mean = ceil_div(s->T * s->k, s->E);
    return mean < s->capacity ? mean : s->capacity;
}

template <typename T>
static bool ffn_fwd(const moe_shape* s, const void* xd, const int32_t* cnt, const void* W1,
                    const void* W2, void* h, void* a, void* yd, float drop_p, uint64_t seed, hipStream_t st) {
    const int E = s->E, C = s->capacity, d = s->d_model, f = s->d_ff;
    const int rows = expected_rows(s);
    GemmArgs p = {};
    p.expert_count = cnt; p.var_k = 0;
    if (drop_p > 0.0f) {
        p.drop_thr = (uint32_t)floor((double)drop_p * 4294967296.0);
        p.drop_scale = (float)(1.0 / (1.0 - (double)drop_p));
        p.seed = seed;
    }
    // z = xd W1 (not stored);  h = act(z), a = act'(z)
    p.A = xd; p.lda = d; p.strideA = (long long)C * d;
    p.B = W1; p.ldb = f; p.strideB = (long long)d * f;
    p.out0 = a; p.out1 = h; p.ldo = f; p.strideO = (long long)C * f;
    p.M = C; p.N = f; p.K = d;
    bool ok;
    if (!a) {   // forward-only: the derivative is neither computed nor stored
        p.out0 = h; p.out1 = nullptr;
        if (s->act == MOE_RELU) ok = launch_gemm<T, true, false, EPI_H, MOE_RELU>(p, rows, E, st);
        else ok = launch_gemm<T, true, false, EPI_H, MOE_GELU>(p, rows, E, st);
    } else if (s->act == MOE_RELU) ok = launch_gemm<T, true, false, EPI_H_DACT, MOE_RELU>(p, rows, E, st);
    else ok = launch_gemm<T, true, false, EPI_H_DACT, MOE_GELU>(p, rows, E, st);
    if (!ok) return false;
    // yd = h W2
    p.A = h; p.lda = f; p.strideA = (long long)C * f;
    p.B = W2; p.ldb = d; p.strideB = (long long)f * d;
    p.out0 = yd; p.out1 = nullptr; p.ldo = d; p.strideO = (long long)C * d;
    p.M = C; p.N = d; p.K = f;
    p.drop_thr = 0;
    return launch_gemm<T, true, false, EPI_STORE>(p, rows, E, st);
}

template <typename T>
static bool ffn_bwd(const moe_shape* s, const void* dyd, const void* xd, const void* h,
                    const void* a, const int32_t* cnt, const void* W1, const void* W2, void* dxd,
                    float* dW1, float* dW2, void* dz, hipStream_t st) {
    const int E = s->E, C = s->capacity, d = s->d_model, f = s->d_ff;
    const int rows = expected_rows(s);
    // Four products in two launches.  dW2 needs only h and dyd, so it shares a launch with dz;
    // dxd and dW1 both need dz and share the second one.
    GemmArgs p = {}, q = {};
    p.expert_count = q.expert_count = cnt;
    // dz = (dyd W2^T) .* a:  B(r = n in f, k in d) = W2[n*d + k]
    p.var_k = 0;
    p.A = dyd; p.lda = d; p.strideA = (long long)C * d;
    p.B = W2; p.ldb = d; p.strideB = (long long)f * d;
    p.out0 = dz; p.aux = a; p.ldo = f; p.strideO = (long long)C * f;
    p.M = C; p.N = f; p.K = d;
    // dW2[f,d] = h^T dyd:  A(r = m in f, k = row) = h[k*f + m], B(r = n in d, k) = dyd[k*d + n]
    q.var_k = 1;
    q.A = h; q.lda = f; q.strideA = (long long)C * f;
    q.B = dyd; q.ldb = d; q.strideB = (long long)C * d;
    q.out0 = dW2; q.ldo = d; q.strideO = (long long)f * d;
    q.M = f; q.N = d; q.K = C;
    q.lead = d + TILE_EPILOGUE;
    if (!launch_gemm_pair<T, true, true, EPI_MUL, false, false, EPI_F32>(p, q, rows, E, st)) return false;
    // dxd = dz W1^T:  B(r = n in d, k in f) = W1[n*f + k]
    p.A = dz; p.lda = f; p.strideA = (long long)C * f;
    p.B = W1; p.ldb = f; p.strideB = (long long)d * f;
    p.out0 = dxd; p.aux = nullptr; p.ldo = d; p.strideO = (long long)C * d;
    p.M = C; p.N = d; p.K = f;
    // dW1[d,f] = xd^T dz
    q.A = xd; q.lda = d; q.strideA = (long long)C * d;
    q.B = dz; q.ldb = f; q.strideB = (long long)C * f;
    q.out0 = dW1; q.ldo = f; q.strideO = (long long)d * f;
    q.M = d; q.N = f; q.K = C;
    q.lead = f + TILE_EPILOGUE;
    return launch_gemm_pair<T, true, true, EPI_STORE, false, false, EPI_F32>(p, q, rows, E, st);
}

// measurement aids: the tile of each of the four launches (xd W1, h W2, dz with dW2, dxd with dW1), and whether it is the
// 32 x 32 one
static int four_tiles(const moe_shape* shape, FfnTile (&t)[4]) {
    int rc = shape_status(shape);
    if (rc || (rc = check_slice_limits(shape))) return rc;
    const bool f32 = shape->dtype == MOE_F32;
    const int rows = expected_rows(shape), d = shape->d_model, f = shape->d_ff, E = shape->E;
    t[0] = tile_for(f32, rows, f, d, E);
    t[1] = tile_for(f32, rows, d, f, E);
    t[2] = tile_for_pair(f32, true, rows, f, f, d, E);
    t[3] = tile_for_pair(f32, false, rows, d, d, f, E);
    return MOE_OK;
}
// and: is every tile of the launch found without the experts' row counts; its workgroups
extern "C" int moe_expert_ffn_direct(const moe_shape* shape, int32_t* direct, int32_t* workgroups) {
    FfnTile t[4];
    const int rc = four_tiles(shape, t);
    if (rc) return rc;
    if (!direct || !workgroups) return MOE_ERR_NULL;
    const bool f32 = shape->dtype == MOE_F32;
    const int d = shape->d_model, f = shape->d_ff;
    for (int i = 0; i < 4; ++i) {
        const int side = t[i] == TILE_32 ? THIN : t[i] == TILE_64 ? 64 : t[i] == TILE_256 ? BIG_M : 128;
        const int occ = t[i] == TILE_32 ? THIN_GRID
            : t[i] == TILE_64 ? (f32 ? MidSmem<float, 64, 64, 2, 2, true, true>::OCC : MidSmem<bf16_t, 64, 64, 1, 3, true, true>::OCC)
            : t[i] == TILE_128_PAIRED ? MidSmem<float, 128, 128, 2, 2, true, true>::OCC
            : f32 ? MidSmem<float, 128, 128, 1, 2, true, true>::OCC : MidSmem<bf16_t, 128, 128, 1, 2, true, true>::OCC;
        GemmArgs p = {}, q = {};
        p.M = shape->capacity;
        p.N = i == 1 || i == 3 ? d : f;
        q.M = i == 2 ? f : d;
        q.N = i == 2 ? d : f;
        set_tiles(p, side, side, shape->E);
        set_tiles(q, side, side, shape->E);
        const int per_xcd = t[i] == TILE_256 ? 0 : set_direct(p, i >= 2 ? &q : nullptr, expected_rows(shape), side, occ);
        direct[i] = per_xcd > 0;
        workgroups[i] = t[i] == TILE_256 ? gemm_grid(all_tiles(p) + (i >= 2 ? all_tiles(q) : 0))
            : per_xcd > 0 ? 8 * per_xcd : mid_grid(p, i >= 2 ? &q : nullptr, occ);
    }
    return MOE_OK;
}
extern "C" int moe_expert_ffn_parts(const moe_shape* shape, int32_t* parts) {
    FfnTile t[4];
    const int rc = four_tiles(shape, t);
    if (rc) return rc;
    if (!parts) return MOE_ERR_NULL;
    for (int i = 0; i < 4; ++i) parts[i] = t[i] == TILE_32;
    return MOE_OK;
}
extern "C" int moe_expert_ffn_tiles(const moe_shape* shape, int32_t* side, int32_t* wave_groups) {
    FfnTile t[4];
    const int rc = four_tiles(shape, t);
    if (rc) return rc;
    if (!side || !wave_groups) return MOE_ERR_NULL;
    const bool f32 = shape->dtype == MOE_F32;
    for (int i = 0; i < 4; ++i) {
        side[i] = t[i] == TILE_32 ? THIN : t[i] == TILE_64 ? 64 : t[i] == TILE_256 ? 256 : 128;
        wave_groups[i] = f32 && (t[i] == TILE_64 || t[i] == TILE_128_PAIRED) ? 2 : 1;
    }
    return MOE_OK;
}

int ffn_fwd_check(const moe_shape* s, const void* xd, const int32_t* expert_count, const void* W1, const void* W2,
                  float drop_p, const void* h_saved, const void* dact_saved, const void* yd) {
    int rc = shape_status(s);
    if (rc || (rc = check_slice_limits(s))) return rc;
    if (!xd || !expert_count || !W1 || !W2 || !h_saved || !yd) return MOE_ERR_NULL;   // dact_saved may be NULL
    if (!(drop_p >= 0.0f && drop_p < 1.0f)) return MOE_ERR_SHAPE;
    return drop_p > 0.0f && !dact_saved ? MOE_ERR_NULL : MOE_OK;      // dropout is a training feature
}

static int ffn_fwd_impl(const moe_shape* shape, const void* xd, const int32_t* expert_count,
                        const void* W1, const void* W2, float drop_p, uint64_t seed, void* h_saved,
                        void* dact_saved, void* yd, void* stream) {
    const int rc = begin_call(ffn_fwd_check(shape, xd, expert_count, W1, W2, drop_p, h_saved, dact_saved, yd));
    if (rc) return rc;
    if (drop_p > 0.0f && floor((double)drop_p * 4294967296.0) < 1.0) drop_p = 0.0f;   // below one part in 2^32
    hipStream_t st = (hipStream_t)stream;
    const bool ok = shape->dtype == MOE_BF16
        ? ffn_fwd<bf16_t>(shape, xd, expert_count, W1, W2, h_saved, dact_saved, yd, drop_p, seed, st)
        : ffn_fwd<float>(shape, xd, expert_count, W1, W2, h_saved, dact_saved, yd, drop_p, seed, st);
    return ok ? launch_status() : MOE_ERR_LAUNCH;
}

extern "C" int moe_expert_ffn_fwd(const moe_shape* shape, const void* xd,
                                  const int32_t* expert_count, const void* W1, const void* W2,
                                  void* h_saved, void* dact_saved, void* yd, void* stream) {
    return ffn_fwd_impl(shape, xd, expert_count, W1, W2, 0.0f, 0, h_saved, dact_saved, yd, stream);
}

extern "C" int moe_expert_ffn_fwd_dropout(const moe_shape* shape, const void* xd,
                                          const int32_t* expert_count, const void* W1, const void* W2,
                                          float drop_p, uint64_t seed, void* h_saved, void* dact_saved,
                                          void* yd, void* stream) {
    return ffn_fwd_impl(shape, xd, expert_count, W1, W2, drop_p, seed, h_saved, dact_saved, yd, stream);
}

int ffn_bwd_check(const moe_shape* s, const void* dyd, const void* xd, const void* h_saved, const void* dact_saved,
                  const int32_t* expert_count, const void* W1, const void* W2, const void* dxd, const float* dW1,
                  const float* dW2, const void* ws, size_t ws_bytes) {
    int rc = shape_status(s);
    if (rc || (rc = check_slice_limits(s))) return rc;
    if (!dyd || !xd || !h_saved || !dact_saved || !expert_count || !W1 || !W2 || !dxd || !dW1 || !dW2)
        return MOE_ERR_NULL;
    return ws_ok(ws, ws_bytes, ffn_bwd_ws_bytes(s)) ? MOE_OK : MOE_ERR_WORKSPACE;
}

extern "C" int moe_expert_ffn_bwd(const moe_shape* shape, const void* dyd, const void* xd,
                                  const void* h_saved, const void* dact_saved,
                                  const int32_t* expert_count, const void* W1, const void* W2,
                                  void* dxd, float* dW1, float* dW2, void* ws, size_t ws_bytes,
                                  void* stream) {
    const int rc = begin_call(ffn_bwd_check(shape, dyd, xd, h_saved, dact_saved, expert_count, W1, W2, dxd, dW1, dW2, ws, ws_bytes));
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    const bool ok = shape->dtype == MOE_BF16
        ? ffn_bwd<bf16_t>(shape, dyd, xd, h_saved, dact_saved, expert_count, W1, W2, dxd, dW1, dW2, ws, st)
        : ffn_bwd<float>(shape, dyd, xd, h_saved, dact_saved, expert_count, W1, W2, dxd, dW1, dW2, ws, st);
    return ok ? launch_status() : MOE_ERR_LAUNCH;
}
