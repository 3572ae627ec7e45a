// fp32 reconstruction GEMMs for gfx950 (v_mfma_f32_32x32x2_f32: fp32 products and sums) with the fused
// MSE and straight-through epilogues.
//
// Bound by the matrix units (256 flop per cycle and CU, twice what separate fp32 FMAs reach without
// packed instructions) once the operands are staged: operand tiles go from memory straight into LDS
// with direct-to-LDS buffer loads, some steps ahead. A workgroup is four waves, each a 32 x 32 tile (16 registers
// per accumulator); three workgroups of 48 KB LDS fit a CU (of the forward's small tile, 65 KB, two), whose waves hide
// each other's waits. 2,037 x 1,001 x 1,504: forward 65 us, backward 73 us with its finishing launch (84 TFLOP/s),
// where 4 x 4 register tiles of scalar FMAs from 4-byte loads took 231 and 253; 128 x 256 x 256: 5.9 and 5.9 us,
// before 42.1 and 22.6.
//
// Operand layout of 32x32x2: lane l holds A[l % 32][l / 32] (resp. B[l / 32][l % 32]); accumulator
// register r of lane l holds C[8 (r / 4) + 4 (l / 32) + r % 4][l % 32]. The reduction index may be
// permuted alike in both operands: the forward's lanes read 16 bytes (4 k) of their row and half, so
// instruction s of a group of 8 k multiplies k = s and k = 4 + s.
#include <type_traits>

#include "gemm_common.h"

namespace focus {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
struct F32Frags {
    f32x4 a[2], b[2];
};

// The fragments of 16 k: reads and their wait in one block, because the compiler would let an LDS read of
// its own wait for every direct-to-LDS load in flight.
__device__ __forceinline__ F32Frags read_frags_f32(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1) {
    F32Frags f;
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %2, %6\n\tds_read_b128 %1, %5\n\tds_read_b128 %3, %7\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f.a[0]), "=&v"(f.a[1]), "=&v"(f.b[0]), "=&v"(f.b[1])
                 : "v"(a0), "v"(a1), "v"(b0), "v"(b1)
                 : "memory");
    return f;
}

// Backward fragments of 16 tokens: rows lh, 2 + lh, .. (256 bytes each) of this lane's column of A and B
// (ds_read2st64_b32 takes two rows, offsets in units of 256 bytes).
struct F32Cols {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    f32x2 a[4], b[4];
};
__device__ __forceinline__ F32Cols read_cols_f32(uint32_t a, uint32_t b) {
    F32Cols f;
    asm volatile("ds_read2st64_b32 %0, %8 offset0:0 offset1:2\n\tds_read2st64_b32 %4, %9 offset0:0 offset1:2\n\t"
                 "ds_read2st64_b32 %1, %8 offset0:4 offset1:6\n\tds_read2st64_b32 %5, %9 offset0:4 offset1:6\n\t"
                 "ds_read2st64_b32 %2, %8 offset0:8 offset1:10\n\tds_read2st64_b32 %6, %9 offset0:8 offset1:10\n\t"
                 "ds_read2st64_b32 %3, %8 offset0:12 offset1:14\n\tds_read2st64_b32 %7, %9 offset0:12 offset1:14\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f.a[0]), "=&v"(f.a[1]), "=&v"(f.a[2]), "=&v"(f.a[3]), "=&v"(f.b[0]), "=&v"(f.b[1]),
                   "=&v"(f.b[2]), "=&v"(f.b[3])
                 : "v"(a), "v"(b)
                 : "memory");
    return f;
}

// ------------------------------------------------------------------------------------------------
// Forward, Y_hat = X_hat W_hat^T (both K-contiguous, K a multiple of 16) with the MSE epilogue or plain.
// Operands are staged as tiles of 64-byte rows (16 k; the layout and swizzle of the bf16 forward).
//   T == 64: 64 x 64 tile, the waves 2 x 2; a step is 32 k (two such tiles per operand), three stages of
//            16 KB, one barrier per step.
//   T == 32: 32 x 32 tile, the waves taking every fourth 16 k each, in four stages of their own (no
//            barrier in the loop). For outputs too small to fill the chip with 64 x 64 tiles: four times the
//            workgroups, a quarter of the serial steps. Each wave keeps four accumulators in turn, so a chain
//            of roundings is K / 16 products long, and the 16 sums are added, and Y_ref subtracted, in fp64. A
//            gradient's largest error comes from the outputs with one very large term, at whose size every
//            later addition rounds: with one accumulator and fp32 sums 1.4e-5 of the gradients' root mean
//            square (128 x 256 x 256, NVFP4, Student-t activations), 2.4e-6 so (5.9 us for 5.4).
template <bool MSE, int T>
__global__ void __launch_bounds__(256)
fwd_f32_kernel(const float *__restrict__ X, const float *__restrict__ W, int64_t M, int64_t N, int64_t K,
               const float *__restrict__ Yref, float *__restrict__ dY, float dscale, double *__restrict__ colpart,
               int tiles_n) {
    constexpr bool kSplit = T == 32;
    constexpr int S = kSplit ? 4 : 3;                     // stages
    constexpr int kSub = T * 64;                          // bytes of one 16-k tile of an operand
    constexpr int kStage = kSplit ? 2 * kSub : 4 * kSub;  // X then W, 16 k or 2 x 16 k each
    constexpr int kLoads = 4;                             // loads per stage per thread
    __shared__ __attribute__((aligned(16))) char smem[kSplit ? 4 * S * kStage : S * kStage];
    __shared__ double red[4][32];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = kSplit ? 0 : wave >> 1, wn = kSplit ? 0 : wave & 1;
    const int lr = lane & 31, lh = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t tm = tile / (uint32_t)tiles_n, tn = tile % (uint32_t)tiles_n;
    const int64_t m0 = tm * T, n0 = tn * T;
    const int64_t pitch = K * 4;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + m0 * K, (M - m0) * pitch);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(W + n0 * K, (N - n0) * pitch);
    // A load instruction fills 1 KB: lane L lands in row L / 4, physical chunk L % 4 of a 16-row group, which
    // holds logical chunk (L % 4) ^ fwd_key(row) (the key depends on row bits 1-3 only).
    const uint32_t lrow = (uint32_t)lane >> 2, chunk = ((uint32_t)lane & 3u) ^ fwd_key(lrow);
    lds_char *const lsm = (lds_char *)smem;
    const int64_t n16 = K / 16;
    const int64_t nk = kSplit ? (n16 + 3 - wave_u) / 4 : (n16 + 1) / 2;  // this wave's steps
    // Slot j of the ring. Loads of k past the row's end (and of slots past the last step) get bit 31 and
    // bring zeros, so every slot is the same number of loads.
    auto issue = [&](int64_t j, int s) {
        lds_char *const st = lsm + (kSplit ? wave_u * S * kStage : 0) + s * kStage;
#pragma unroll
        for (int i = 0; i < kLoads; i++) {
            // T == 64: this wave's 16 rows of X k-tile 0, 1, then of W's; T == 32: rows 0-15, 16-31 of X, then W
            const int op = i >> 1, h = i & 1;
            const int64_t k16 = kSplit ? 4 * j + wave_u : 2 * j + h;
            const uint32_t row = (kSplit ? (uint32_t)h * 16u : (uint32_t)wave_u * 16u) + lrow;
            const uint32_t off = (row * (uint32_t)pitch + (uint32_t)k16 * 64u + chunk * 16u) |
                                 (k16 < n16 ? 0u : 0x80000000u);
            lds_char *const dst = kSplit ? st + op * kSub + h * 1024 : st + (2 * op + h) * kSub + wave_u * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(op ? rw : rx, dst, 16, (int)off, 0, 0, 0);
        }
    };
    constexpr int kAcc = kSplit ? 4 : 1;  // accumulators, taking the instructions in turn
    f32x16_t acc[kAcc] = {};
    // this lane's 16-byte chunks lh and 2 + lh of its rows of a 16-k tile of A and B
    const uint32_t lds0 = (uint32_t)(uintptr_t)lsm + (kSplit ? (uint32_t)wave_u * S * kStage : 0u);
    const uint32_t a0 = fwd_off(wm * 32 + lr, lh), a1 = fwd_off(wm * 32 + lr, 2 + lh);
    const uint32_t b0 = fwd_off(wn * 32 + lr, lh), b1 = fwd_off(wn * 32 + lr, 2 + lh);
    auto mma = [&](uint32_t as, uint32_t bs) {
        const F32Frags f = read_frags_f32(as + a0, as + a1, bs + b0, bs + b1);
#pragma unroll
        for (int e = 0; e < 8; e++)
            acc[e % kAcc] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[e / 4][e % 4], f.b[e / 4][e % 4], acc[e % kAcc], 0, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < S - 1; s++) issue(s, s);
    int sc = 0;
    for (int64_t kt = 0; kt < nk; kt++) {
        FOCUS_WAIT_VMCNT(kLoads * (S - 2));  // this thread's loads of slot kt have landed
        if constexpr (!kSplit) asm volatile("s_barrier" ::: "memory");
        else asm volatile("" ::: "memory");
        const uint32_t st = lds0 + (uint32_t)sc * kStage;
        // after the barrier every wave is done with the stage before, which slot kt + S - 1 refills (T == 32:
        // this wave's own reads of it have returned: its instructions used them)
        const int sp = sc == 0 ? S - 1 : sc - 1;
        issue(kt + S - 1, sp);
        if constexpr (kSplit) {
            mma(st, st + kSub);
        } else {
            mma(st, st + 2 * kSub);
            mma(st + kSub, st + 3 * kSub);
        }
        sc = sc == S - 1 ? 0 : sc + 1;
    }
    // the empty slots' zero writes must land before their LDS is used again or handed on
    FOCUS_WAIT_VMCNT(0);
    __syncthreads();
    // ---- epilogue: this wave's registers r0 .. r0 + R - 1 of the tile's accumulator ----
    constexpr int R = kSplit ? 4 : 16;
    typename std::conditional<kSplit, double, float>::type o[R];
    if constexpr (kSplit) {
        double *part = reinterpret_cast<double *>(smem);  // [wave][register][lane]
#pragma unroll
        for (int r = 0; r < 16; r++)
            part[(wave * 16 + r) * 64 + lane] = ((double)acc[0][r] + (double)acc[1][r]) + ((double)acc[2][r] + (double)acc[3][r]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; r++) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < 4; w++) s += part[(w * 16 + wave * 4 + r) * 64 + lane];
            o[r] = s;
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; r++) o[r] = acc[0][r];
    }
    const int64_t n = n0 + wn * 32 + lr;
    const bool n_ok = n < N;
    double csum = 0.0;
    float y[R];
    auto row_of = [&](int r) { return m0 + wm * 32 + (kSplit ? 8 * wave + r : 8 * (r / 4) + r % 4) + 4 * lh; };
    if constexpr (MSE) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t m = row_of(r);
            y[r] = n_ok && m < M ? Yref[m * N + n] : 0.0f;
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int64_t m = row_of(r);
        if (n_ok && m < M) {
            if constexpr (MSE) {
                const float d = (float)(o[r] - y[r]);
                dY[m * N + n] = d * dscale;
                csum += (double)d * (double)d;
            } else {
                dY[m * N + n] = (float)o[r];
            }
        }
    }
    if constexpr (!MSE) return;
    csum += __shfl_xor(csum, 32, 64);
    if (lh == 0) red[wave][lr] = csum;
    __syncthreads();
    if (t < T && n0 + t < N) {
        double s;
        if constexpr (kSplit) s = ((red[0][t] + red[1][t]) + red[2][t]) + red[3][t];
        else s = red[t >> 5][t & 31] + red[2 + (t >> 5)][t & 31];
        colpart[tm * N + n0 + t] = s;
    }
}

// ------------------------------------------------------------------------------------------------
// Backward, G = dY^T X_hat over the tokens of one split (both token-major), 64 n x 64 k per workgroup, the
// waves 2 x 2, with the fused straight-through epilogue. A step is 32 tokens ([32][64] floats per operand,
// three stages of 16 KB); fragments are 4-byte LDS reads of 32 consecutive columns. dY rows start on 4-byte
// boundaries only unless N % 4 == 0: they are then staged with 4-byte loads (W16 == false).
// A chain of roundings is 64 tokens long, the chains are added in fp64: with one chain per split the gradients'
// error against 64 bits was up to 4.4 times that of many short splits (3,507 x 1,758 x 160: 3.1e-7 for 7.0e-8; now
// 6.4e-8). The additions run beside the next chain's matrix instructions (3,507 x 1,758 x 160 36.9 us for 37.5,
// 4,096 x 2,048 x 2,048 316 for 306); chains of 32 tokens took 41 and 347, of 128 left some errors above.
template <int FMT, int WDT, bool W16>
__global__ void __launch_bounds__(256)
bwd_f32_kernel(const float *__restrict__ dY, const float *__restrict__ X, int64_t M, int64_t N, int64_t K, int64_t chunk,
               const void *__restrict__ W, const float *__restrict__ s_fp, const float *__restrict__ c, int sb_log2,
               const float *__restrict__ alpha_ptr, int ste_clip, int e8m0_floor, float *__restrict__ part_s,
               float *__restrict__ part_c, int direct, float *__restrict__ G_out, uint32_t *flag, int tiles_k) {
        constexpr int T = kF32Tile, kStep = kF32TokenStep, S = 3;
    constexpr int kOp = kStep * T * 4, kStage = 2 * kOp;  // 8 KB per operand
    constexpr int kLoadsY = W16 ? 2 : 8, kLoads = kLoadsY + 2;
    __shared__ __attribute__((aligned(16))) char smem[S * kStage];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31, lh = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t tiles = gridDim.x, id = xcd_tile(blockIdx.y * tiles + blockIdx.x, tiles * gridDim.y);
    const int64_t split = id / tiles;
    const uint32_t tile = id % tiles;
    const int64_t n0 = (int64_t)(tile / (uint32_t)tiles_k) * T, k0 = (int64_t)(tile % (uint32_t)tiles_k) * T;
    const int64_t t_begin = split * chunk, t_end = std::min<int64_t>(M, t_begin + chunk);
    const int64_t nk = t_end > t_begin ? (t_end - t_begin + kStep - 1) / kStep : 0;
    lds_char *const lsm = (lds_char *)smem;
    // A 16-byte load instruction fills 4 token rows (lane L: row L / 16, columns 4 (L % 16) .. + 3), a 4-byte
    // one a single row. Columns past the matrix get bit 31 and read as zeros; rows past the token range lie
    // outside the step's resource.
    const uint32_t row16 = (uint32_t)lane >> 4, col16 = 4u * ((uint32_t)lane & 15u);
    const uint32_t x_bad = (uint32_t)(k0 + col16 >= K) << 31;
    const uint32_t y_bad = (uint32_t)(n0 + (W16 ? col16 : (uint32_t)lane) >= N) << 31;
    auto issue = [&](int64_t j, int s) {
        const int64_t t0 = t_begin + j * kStep, rem = t_end - t0;
        const int64_t rows = rem <= 0 ? 0 : (rem < kStep ? rem : kStep);
        const __amdgpu_buffer_rsrc_t ry = make_rsrc(dY + (rows ? t0 * N : 0), rows * N * 4);
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + (rows ? t0 * K : 0), rows * K * 4);
        lds_char *const st = lsm + s * kStage;
#pragma unroll
        for (int i = 0; i < kLoadsY; i++) {
            if constexpr (W16) {
                const uint32_t blk = (uint32_t)wave_u * 2u + i, row = 4u * blk + row16;
                const uint32_t off = ((row * (uint32_t)N + (uint32_t)n0 + col16) * 4u) | y_bad;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ry, st + blk * 1024, 16, (int)off, 0, 0, 0);
            } else {
                const uint32_t row = (uint32_t)wave_u * 8u + i;
                const uint32_t off = ((row * (uint32_t)N + (uint32_t)n0 + (uint32_t)lane) * 4u) | y_bad;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ry, st + row * 256, 4, (int)off, 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const uint32_t blk = (uint32_t)wave_u * 2u + i, row = 4u * blk + row16;
            const uint32_t off = ((row * (uint32_t)K + (uint32_t)k0 + col16) * 4u) | x_bad;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, st + kOp + blk * 1024, 16, (int)off, 0, 0, 0);
        }
    };
    f32x16_t acc0 = {}, acc1 = {};  // one collects two steps while the other's sums go to gsum, half of them per step
    double gsum[16] = {};
    auto fold = [&](const f32x16_t &a, int half) {
#pragma unroll
        for (int r = 8 * half; r < 8 * half + 8; r++) gsum[r] += (double)a[r];
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)lsm;
    const uint32_t a_off = (uint32_t)(lh * T + wm * 32 + lr) * 4u, b_off = (uint32_t)(lh * T + wn * 32 + lr) * 4u;
#pragma unroll
    for (int s = 0; s < S - 1; s++) issue(s, s);
    int sc = 0;
    auto step = [&](auto half, int64_t kt, f32x16_t &acc, const f32x16_t &before) {
        FOCUS_WAIT_VMCNT(kLoads * (S - 2));
        asm volatile("s_barrier" ::: "memory");
        const uint32_t as = lds0 + (uint32_t)sc * kStage, bs = as + kOp;
        issue(kt + S - 1, sc == 0 ? S - 1 : sc - 1);  // the stage that every wave was done with at the barrier
        if (half == 0) acc = f32x16_t{};
#pragma unroll
        for (int h = 0; h < kStep / 16; h++) {
            const F32Cols f = read_cols_f32(as + a_off + h * 16 * T * 4, bs + b_off + h * 16 * T * 4);
#pragma unroll
            for (int s = 0; s < 8; s++)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[s / 2][s % 2], f.b[s / 2][s % 2], acc, 0, 0, 0);
            if (h == 0) fold(before, half);
        }
        sc = sc == S - 1 ? 0 : sc + 1;
    };
    constexpr std::integral_constant<int, 0> lo{};
    constexpr std::integral_constant<int, 1> hi{};
    int64_t kt = 0;
    for (; kt + 4 <= nk; kt += 4) {
        step(lo, kt, acc0, acc1);
        step(hi, kt + 1, acc0, acc1);
        step(lo, kt + 2, acc1, acc0);
        step(hi, kt + 3, acc1, acc0);
    }
    fold(acc1, 0), fold(acc1, 1);
    acc1 = f32x16_t{};
    if (kt + 2 <= nk) {
        step(lo, kt, acc0, acc1);
        step(hi, kt + 1, acc0, acc1);
        fold(acc0, 0), fold(acc0, 1);
        kt += 2;
    }
    if (kt < nk) {
        step(lo, kt, acc0, acc1);
        fold(acc0, 0), fold(acc0, 1);
    }
    FOCUS_WAIT_VMCNT(0);  // the empty slots' zero writes
    __syncthreads();
    // ---- G to LDS, then pieces of 8 consecutive k of one row per thread (see ste_piece) ----
    constexpr int kPitch = T + 4;
    float *const Gs = reinterpret_cast<float *>(smem);  // [64][68]
#pragma unroll
    for (int r = 0; r < 16; r++)
        Gs[(wm * 32 + 8 * (r / 4) + 4 * lh + r % 4) * kPitch + wn * 32 + lr] = (float)gsum[r];
    __syncthreads();
    constexpr int B = block_of(FMT);
    const float alpha = FMT == kFmtNV ? *alpha_ptr : 1.0f;
    const int64_t nb = K / B, ns = K >> sb_log2;
    bool bad = false;
    auto pieces = [&](auto nc) {
        constexpr int NCOEF = decltype(nc)::value;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int r = (t >> 3) + 32 * i, kc = (t & 7) * 8;
            const int64_t n = n0 + r, k = k0 + kc;
            const bool ok = n < N && k < K;
            float g[8], w[8] = {}, cw[NCOEF], sv = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; e++) g[e] = Gs[r * kPitch + kc + e];
#pragma unroll
            for (int j = 0; j < NCOEF; j++) cw[j] = 1.0f;
            if (ok) {
                load8(W, WDT, n * K + k, w);
                sv = s_fp[n * nb + k / B];
                if (c) {
#pragma unroll
                    for (int j = 0; j < NCOEF; j++) cw[j] = c[n * ns + (k >> sb_log2) + j];
                }
            }
            bool fast = true, nan = false;
#pragma unroll
            for (int e = 0; e < 8; e++) fast = fast && __builtin_fabsf(w[e]) <= 0x1p80f;
            uint32_t byte;
            const float sdq = weight_sdq(FMT, sv, alpha, e8m0_floor, byte, nan);
#pragma unroll
            for (int j = 0; j < NCOEF; j++) nan = nan || bad_coeff(cw[j]);
            bad = bad || (ok && nan);
            float tc[NCOEF], ts;
            ste_piece<NCOEF>(g, w, sdq, cw, fast, ok, ste_clip, tc, ts);
            if constexpr (NCOEF == 1) {
                if (sb_log2 >= 4) tc[0] += quad_xor<1>(tc[0]);
                if (sb_log2 >= 5) tc[0] += quad_xor<2>(tc[0]);
            }
            ts += quad_xor<1>(ts);
            if (B == 32) ts += quad_xor<2>(ts);
            if (FMT == kFmtNV && direct) ts *= alpha;
            if (!ok) continue;
            if (NCOEF > 1 || (kc & ((1 << sb_log2) - 1)) == 0) {
#pragma unroll
                for (int j = 0; j < NCOEF; j++)
                    part_c[(split * N + n) * ns + (k >> sb_log2) + j] = direct ? -tc[j] / (cw[j] * cw[j]) : tc[j];
            }
            if ((kc & (B - 1)) == 0) part_s[(split * N + n) * nb + k / B] = ts;
            if (G_out) {
#pragma unroll
                for (int e = 0; e < 8; e++) G_out[n * K + k + e] = g[e];
            }
        }
    };
    if (sb_log2 >= 3) pieces(std::integral_constant<int, 1>{});
    else if (sb_log2 == 2) pieces(std::integral_constant<int, 2>{});
    else pieces(std::integral_constant<int, 4>{});
    if (bad) raise_domain_flag(flag);
}

}  // namespace

// Buffer offsets are 32-bit: a tile's rows must span less than 2^31 bytes. The tiles make a one-dimensional grid, whose
// work-items (256 per tile) must stay below 2^32.
static bool f32_grid_fits(int64_t rows, int64_t cols) {
    return ((rows + kF32Tile - 1) / kF32Tile) * ((cols + kF32Tile - 1) / kF32Tile) < (int64_t(1) << 24);
}

bool f32_fwd_supported(int64_t M, int64_t N, int64_t K) {
    return K % 16 == 0 && int64_t(kF32Tile) * K * 4 < (int64_t(1) << 31) && f32_grid_fits(M, N);
}

bool f32_bwd_supported(int64_t M, int64_t N, int64_t K) {
    (void)M;
    return int64_t(kF32TokenStep) * N * 4 < (int64_t(1) << 31) && int64_t(kF32TokenStep) * K * 4 < (int64_t(1) << 31) &&
           f32_grid_fits(N, K);
}

hipError_t launch_fwd_f32(int tile, const float *X, const float *W, int64_t M, int64_t N, int64_t K, const float *Yref,
                          float *dY, float dscale, double *colpart, hipStream_t st) {
    const int tiles_n = (int)((N + tile - 1) / tile);
    const dim3 grid((unsigned)((M + tile - 1) / tile) * tiles_n);
#define FF(MSE, T) fwd_f32_kernel<MSE, T><<<grid, 256, 0, st>>>(X, W, M, N, K, Yref, dY, dscale, colpart, tiles_n)
    if (tile == kF32Tile) { if (Yref) FF(true, 64); else FF(false, 64); }
    else { if (Yref) FF(true, 32); else FF(false, 32); }
#undef FF
    return hipGetLastError();
}

hipError_t launch_bwd_f32(int fmt, int w_dt, const float *dY, const float *X, int64_t M, int64_t N, int64_t K,
                          int64_t chunk, int64_t splits, const void *W, const float *s_fp, const float *c, int sb,
                          const float *alpha, int ste_clip, int e8m0_floor, float *part_s, float *part_c, int direct,
                          float *G_out, uint32_t *flag, hipStream_t st) {
    const int tiles_n = (int)((N + kF32Tile - 1) / kF32Tile), tiles_k = (int)((K + kF32Tile - 1) / kF32Tile);
    int sbl = 0;
    while ((1 << sbl) < sb) sbl++;
    const dim3 grid((unsigned)tiles_n * tiles_k, (unsigned)splits);
#define BF(F, WD, V) bwd_f32_kernel<F, WD, V><<<grid, 256, 0, st>>>(dY, X, M, N, K, chunk, W, s_fp, c, sbl, alpha, ste_clip, e8m0_floor, part_s, part_c, direct, G_out, flag, tiles_k)
#define BF_V(F, WD) if (N % 4 == 0) BF(F, WD, true); else BF(F, WD, false)
    if (fmt == kFmtMX) { if (w_dt == kBF16) { BF_V(kFmtMX, kBF16); } else { BF_V(kFmtMX, kF32); } }
    else { if (w_dt == kBF16) { BF_V(kFmtNV, kBF16); } else { BF_V(kFmtNV, kF32); } }
#undef BF_V
#undef BF
    return hipGetLastError();
}

}  // namespace focus
