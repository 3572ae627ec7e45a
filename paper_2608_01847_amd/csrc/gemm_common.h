// Pieces shared by the VALU and MFMA reconstruction GEMMs.
#pragma once

#include "focus_device.h"

#include <algorithm>
#include <utility>

namespace focus {

__device__ __forceinline__ float load1(const void *base, int dtype, int64_t i) {
    return dtype == kBF16 ? bf16_bits_to_f32(reinterpret_cast<const uint16_t *>(base)[i])
                          : reinterpret_cast<const float *>(base)[i];
}

__device__ __forceinline__ void store1(void *base, int dtype, int64_t i, float v) {
    if (dtype == kBF16) reinterpret_cast<uint16_t *>(base)[i] = (uint16_t)f32_to_bf16_bits(v);
    else reinterpret_cast<float *>(base)[i] = v;
}

// Straight-through terms of one weight element given g = dL/dW_hat (Sec. 3.2 STE through Eq. 6-8):
// W_hat = Q(w / (S_dq c)) S_dq with Q -> clamp, so dW_hat/dc = -m w / c^2 and
// dW_hat/dS_dq = q - m u. The caller sums tc over the sub-block (then scales by -1/c^2) and ts over
// the block.
__device__ __forceinline__ void ste_terms(float g, float w, float sdq, float cval, bool ste_clip,
                                          float &tc, float &ts) {
    Quantized z = quantize_element(w, sdq * cval, sdq, ste_clip);
    tc = z.m ? g * w : 0.0f;
    ts = g * (z.q - (z.m ? z.u : 0.0f));
}

typedef float f32x16_t __attribute__((ext_vector_type(16)));

// Raw buffer resources: a load whose offset is at or past num_records returns zeros and a store
// there is dropped, so bounds are handled by the hardware range check instead of branches (an
// offset with bit 31 set is always past it, since num_records is kept below 2^31).
constexpr int kRsrcWord3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int64_t bytes) {
    const int64_t n = bytes < 0 ? 0 : (bytes > 0x7FFFFFFF ? 0x7FFFFFFF : bytes);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)n, kRsrcWord3);
}

typedef __attribute__((address_space(3))) char lds_char;

// Row `row`'s xor key for the 64-byte-row tile: ((row >> 1) & 3) ^ ((row >> 3) & 1). A fragment
// read serves 8 or 16 consecutive rows of one logical chunk per cycle; with this key those rows
// land on distinct 16-byte slots of a 128- or 256-byte bank span.
__device__ __forceinline__ uint32_t fwd_key(uint32_t row) { return ((row >> 1) & 3u) ^ ((row >> 3) & 1u); }

// Byte offset of 16-byte chunk `chunk` (0..3) of row `row` in a 64-byte-row tile.
__device__ __forceinline__ uint32_t fwd_off(uint32_t row, uint32_t chunk) {
    return row * 64u + ((chunk ^ fwd_key(row)) << 4);
}

// s_waitcnt with vmcnt <= n (n < 64) and the LDS and export counters unconstrained
#define FOCUS_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))

// Workgroups are dealt to the 8 XCDs round-robin (id % 8), each XCD with its own L2. Renumbering
// so that XCD x runs a contiguous block of tiles keeps tiles that share operand panels in one L2.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t id, uint32_t count) {
    const uint32_t per = count / 8u;
    return id < per * 8u ? (id % 8u) * per + id / 8u : id;
}

// Calls f(std::integral_constant<int, 0>) ... f(<N-1>): every accumulator index is then a
// compile-time constant, so the accumulators stay in registers.
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// the value of lane l ^ X (X = 1 or 2), a DPP move within each four lanes
template <int X>
__device__ __forceinline__ float quad_xor(float v) {
    constexpr int kCtrl = X == 1 ? 0xB1 : 0x4E;  // quad_perm [1, 0, 3, 2] / [2, 3, 0, 1]
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), kCtrl, 0xF, 0xF, true));
}

// The straight-through sums of 8 consecutive elements of one row, NCOEF coefficients among them:
// tc[j] = sum of G m w over coefficient j's elements, ts = sum of G (q - m u). u comes from one
// correctly rounded reciprocal per coefficient where the whole wave's operands are in div_by_scale's
// range (`fast`; lanes with !ok, whose sums the caller drops, do not count), else from a true division.
template <int NCOEF>
__device__ __forceinline__ void ste_piece(const float (&g)[8], const float (&w)[8], float sdq, const float (&cw)[NCOEF],
                                          bool fast, bool ok, int ste_clip, float (&tc)[NCOEF], float &ts) {
    constexpr int EPC = 8 / NCOEF;  // elements per coefficient
    ts = 0.0f;
#pragma unroll
    for (int k = 0; k < NCOEF; k++) {
        tc[k] = 0.0f;
        fast = fast && scale_in_fast_range(sdq * cw[k]);
    }
    if (__builtin_expect(__all(fast || !ok), 1)) {
        const float lim = ste_clip ? 6.0f : __builtin_inff();
        float u[8], qv[8];
#pragma unroll
        for (int k = 0; k < NCOEF; k++) {
            const float sq = sdq * cw[k], y = 1.0f / sq;
#pragma unroll
            for (int e = k * EPC; e < (k + 1) * EPC; e++) u[e] = div_by_scale(w[e], sq, y);
        }
        uint32_t p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, u[0], u[1], 1.0f, 0);
        p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, u[2], u[3], 1.0f, 1);
        p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, u[4], u[5], 1.0f, 2);
        p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, u[6], u[7], 1.0f, 3);
        e2m1_value2<0>(p, qv[0], qv[1]);
        e2m1_value2<1>(p, qv[2], qv[3]);
        e2m1_value2<2>(p, qv[4], qv[5]);
        e2m1_value2<3>(p, qv[6], qv[7]);
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const bool m = __builtin_fabsf(u[e]) <= lim;
            tc[e / EPC] = m ? __builtin_fmaf(g[e], w[e], tc[e / EPC]) : tc[e / EPC];
            ts = __builtin_fmaf(g[e], qv[e] - (m ? u[e] : 0.0f), ts);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; e++) {
            float a1, a2;
            ste_terms(g[e], w[e], sdq, cw[e / EPC], ste_clip != 0, a1, a2);
            tc[e / EPC] += a1;
            ts += a2;
        }
    }
}

// ---- fp32 MFMA path (gemm_f32.hip) --------------------------------------------------------------
constexpr int kF32Tile = 64;        // output tile edge (the forward's small tile: half of it)
constexpr int kF32TokenStep = 32;   // backward reduction step over tokens

bool f32_fwd_supported(int64_t M, int64_t N, int64_t K);
bool f32_bwd_supported(int64_t M, int64_t N, int64_t K);
// `tile` is kF32Tile or kF32Tile / 2, rows of a colpart row likewise
hipError_t launch_fwd_f32(int tile, const float *X, const float *W, int64_t M, int64_t N, int64_t K, const float *Yref,
                          float *dY, float dscale, double *colpart, hipStream_t st);
// With `direct` (splits == 1) part_s / part_c are the gradients themselves; G_out (splits == 1) may be NULL.
hipError_t launch_bwd_f32(int fmt, int w_dt, const float *dY, const float *X, int64_t M, int64_t N, int64_t K,
                          int64_t chunk, int64_t splits, const void *W, const float *s_fp, const float *c, int sb,
                          const float *alpha, int ste_clip, int e8m0_floor, float *part_s, float *part_c, int direct,
                          float *G_out, uint32_t *flag, hipStream_t st);

// ---- MFMA path geometry (gemm_mfma.hip) -------------------------------------------------------
constexpr int kMfmaTileM = 256;       // forward output tile: tokens
constexpr int kMfmaTileN = 256;       // backward output tile: out features
constexpr int kMfmaTileK = 256;       // backward output tile: in features
constexpr int kMfmaTokenStep = 64;    // backward reduction step over tokens
constexpr int kMfmaConcurrentWgs = 256;  // one 128 KB-LDS workgroup per CU, 256 CUs

constexpr int kSmallTile = 128;       // both tile edges of the small-tile kernels (gemm_small.hip)

bool mfma_fwd_supported(int64_t M, int64_t N, int64_t K);
bool mfma_bwd_supported(int64_t M, int64_t N, int64_t K);
hipError_t launch_fwd_mfma(const void *X, const void *W, int64_t M, int64_t N, int64_t K, const void *Yref,
                           void *dY, float dscale, double *colpart, hipStream_t st);
// the forward on 128 x 128 tiles: bf16 operands (Xs == nullptr) or packed MXFP4
hipError_t launch_fwd_small(const void *X, const void *W, const void *Xs, const void *Ws, int64_t M, int64_t N, int64_t K,
                            const void *Yref, void *dY, float dscale, double *colpart, hipStream_t st);
// the backward on 128 x 128 tiles: X is bf16 X_hat (Xs == nullptr) or the packed MXFP4 codes
hipError_t launch_bwd_small(int fmt, int w_dt, const void *dY, const void *X, const void *Xs, int64_t M, int64_t N, int64_t K,
                            int64_t chunk, int64_t splits, const void *W, const float *s_fp, const float *c, int sb,
                            const float *alpha, int ste_clip, int e8m0_floor, float *part_s, float *part_c, int direct,
                            uint32_t *flag, hipStream_t st);
// dX_hat = dY W_hat (bf16); with splits > 1 through `splits` x [M][K] fp32 sums in `part`
bool mfma_dx_supported(int64_t M, int64_t N, int64_t K);
hipError_t launch_dx_mfma(const void *dY, const void *W, int64_t M, int64_t N, int64_t K, int64_t chunk, int64_t splits,
                          void *dX, float *part, hipStream_t st);
// the same product from packed MXFP4 operands (X codes [M][K/2], W codes in K-slabs [K/128][N][64],
// block-major E8M0 bytes [K/32][rows]; K % 128 == 0)
bool mfma_fwd_mx_supported(int64_t M, int64_t N, int64_t K);
hipError_t launch_fwd_mfma_mx(const void *Xc, const void *Xs, const void *Wc, const void *Ws, int64_t M, int64_t N,
                              int64_t K, const void *Yref, void *dY, float dscale, double *colpart, hipStream_t st);
// The fused backward. With `direct` (splits == 1) part_s / part_c are the gradients themselves.
hipError_t launch_bwd_mfma(int fmt, int w_dt, const void *dY, const void *X, int64_t M, int64_t N, int64_t K,
                           int64_t chunk, int64_t splits, const void *W, const float *s_fp, const float *c,
                           int sb, const float *alpha, int ste_clip, int e8m0_floor, float *part_s,
                           float *part_c, int direct, uint32_t *flag, hipStream_t st);

// the backward from X_hat as packed MXFP4 (codes [M][K/2], E8M0 bytes block-major [K/32][M])
bool mfma_bwd_mx_supported(int64_t M, int64_t N, int64_t K);
hipError_t launch_bwd_mfma_mx(int w_dt, const void *dY, const void *Xc, const void *Xs, int64_t M, int64_t N,
                              int64_t K, int64_t chunk, int64_t splits, const void *W, const float *s_fp,
                              const float *c, int sb, int ste_clip, int e8m0_floor, float *part_s, float *part_c,
                              int direct, uint32_t *flag, hipStream_t st);

}  // namespace focus
