// The bf16 / packed-MXFP4 reconstruction GEMMs on 128 x 128 tiles, for layers and batches whose 256 x 256 tiles
// leave most CUs without one. Same operands, instructions and per-element order of sums as the kernels of
// gemm_mfma.hip; a workgroup is four waves, 2 x 2, each owning 64 x 64 (2 x 2 MFMA tiles of 32 x 32), and two
// workgroups share a CU, whose waves hide each other's waits for LDS and memory, so the pipeline is a plain one:
// wait for the step's slot, barrier, read fragments, refill the stage before, multiply. Bound by the operands' way
// from L2 (a 128 x 128 tile moves twice the bytes per product: 16 KB per step and CU take 0.38 us, 11 TB/s over the
// chip, whatever the depth of the ring).
#include "mfma_common.h"

namespace focus {

namespace {

constexpr int kT = kSmallTile;  // output tile edge
constexpr int kThreads = 256;

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// A step's fragments: rows + 0 and + 32 of the wave's 64, for both half-steps; MXFP4: the scale words of the same
// rows in blocks lh and 2 + lh. The reads and their wait are one block, because the compiler would let an LDS read
// of its own wait for every direct-to-LDS load in flight.
struct FwdStepFrags {
    bf16x8_t a[2][2], b[2][2];  // [half][rows]
    u32x2_t x[2], w[2];
};

__device__ __forceinline__ void read_step(FwdStepFrags &f, uint32_t a0, uint32_t b0, uint32_t a1, uint32_t b1) {
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %4, %9\n\tds_read_b128 %1, %8 offset:2048\n\t"
                 "ds_read_b128 %5, %9 offset:2048\n\tds_read_b128 %2, %10\n\tds_read_b128 %6, %11\n\t"
                 "ds_read_b128 %3, %10 offset:2048\n\tds_read_b128 %7, %11 offset:2048\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(f.a[0][0]), "=&v"(f.a[0][1]), "=&v"(f.a[1][0]), "=&v"(f.a[1][1]), "=&v"(f.b[0][0]),
                   "=&v"(f.b[0][1]), "=&v"(f.b[1][0]), "=&v"(f.b[1][1])
                 : "v"(a0), "v"(b0), "v"(a1), "v"(b1)
                 : "memory");
}

__device__ __forceinline__ void read_step_mx(FwdStepFrags &f, uint32_t a0, uint32_t b0, uint32_t a1, uint32_t b1,
                                             uint32_t x, uint32_t w) {
    asm volatile("ds_read_b64 %8, %16\n\tds_read_b64 %9, %16 offset:256\n\tds_read_b64 %10, %17\n\t"
                 "ds_read_b64 %11, %17 offset:256\n\t"
                 "ds_read_b128 %0, %12\n\tds_read_b128 %4, %13\n\tds_read_b128 %1, %12 offset:2048\n\t"
                 "ds_read_b128 %5, %13 offset:2048\n\tds_read_b128 %2, %14\n\tds_read_b128 %6, %15\n\t"
                 "ds_read_b128 %3, %14 offset:2048\n\tds_read_b128 %7, %15 offset:2048\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(f.a[0][0]), "=&v"(f.a[0][1]), "=&v"(f.a[1][0]), "=&v"(f.a[1][1]), "=&v"(f.b[0][0]),
                   "=&v"(f.b[0][1]), "=&v"(f.b[1][0]), "=&v"(f.b[1][1]), "=&v"(f.x[0]), "=&v"(f.x[1]), "=&v"(f.w[0]),
                   "=&v"(f.w[1])
                 : "v"(a0), "v"(b0), "v"(a1), "v"(b1), "v"(x), "v"(w)
                 : "memory");
}

// ------------------------------------------------------------------------------------------------
// Forward (see fwd_mfma_kernel): 64 bytes of each operand row per step, four stages of 16 KB (17 KB for MXFP4).
// 2,048 x 1,024 x 2,560: MXFP4 16.9 us, bf16 34.5 us with the two finishing kernels; on 256 x 256 tiles 29.4 and 62.7.
template <bool MSE, bool MX, bool WIDE>
__global__ void __launch_bounds__(kThreads, 2)
fwd_small_kernel(const void *__restrict__ X, const void *__restrict__ W, const uint8_t *__restrict__ Xs,
                 const uint8_t *__restrict__ Ws, int64_t M, int64_t N, int64_t K, const uint16_t *__restrict__ Yref,
                 uint16_t *__restrict__ dY, float dscale, double *__restrict__ colpart, int tiles_n, int group) {
    constexpr int S = 4, kOp = kT * 64, kStage = 2 * kOp + (MX ? 1024 : 0);
    constexpr int kLoads = MX ? 5 : 4;     // loads per slot per thread
    constexpr int kKStep = MX ? 128 : 32;  // k per step
    __shared__ __attribute__((aligned(16))) char smem[S * kStage];
    __shared__ double red[2][kT];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31, lh = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    uint32_t tm, tn;
    if constexpr (!WIDE) tm = tile / (uint32_t)tiles_n, tn = tile % (uint32_t)tiles_n;
    else grouped_tile(tile, gridDim.x / (uint32_t)tiles_n, (uint32_t)tiles_n, tm, tn, (uint32_t)group);
    const int64_t m0 = (int64_t)tm * kT, n0 = (int64_t)tn * kT;
    const int64_t pitch = MX ? K / 2 : K * 2;
    const int64_t nk = (K + kKStep - 1) / kKStep;
    lds_char *const lsm = (lds_char *)smem;
    FwdDma<2> dma, dmaw;  // dmaw: MXFP4 weight codes, rows of 64 bytes in K-slab j
    dma.init(pitch, wave_u, lane);
    dmaw.init(64, wave_u, lane);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(static_cast<const char *>(X) + m0 * pitch, (M - m0) * pitch);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(static_cast<const char *>(W) + n0 * pitch, (N - n0) * pitch);
    const char *const ws_base = static_cast<const char *>(W) + n0 * 64;
    const int64_t w_slab = N * 64;
    // Scale bytes: per stage [4 blocks][128 rows] of X, then of W. Wave w brings blocks 2 (w % 2) and + 1 of X (w < 2)
    // or W; lane L's 4 bytes land at word L % 32 of block L / 32, word (8 h + a) 2 + i holding rows 64 h + 32 i + 4 a
    // .. + 3, so that a fragment lane's rows lr and 32 + lr lie in adjacent words.
    const int64_t s_rows = wave_u < 2 ? M : N;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(wave_u < 2 ? Xs : Ws, MX ? (K / 32) * s_rows : 0);
    const uint32_t sp = (uint32_t)lane & 31u;
    const uint32_t s_row = (uint32_t)(wave_u < 2 ? m0 : n0) + (sp >> 4) * 64u + (sp & 1u) * 32u + ((sp >> 1) & 7u) * 4u;
    auto issue = [&](int64_t j, int s) {
        lds_char *const st = lsm + s * kStage;
        const uint32_t off = j < nk ? 0u : 0x80000000u;  // slots past the last step bring zeros
        const uint32_t base = (uint32_t)j * 64u, bad = dma.step_bad(pitch, (int64_t)j * 64) | off;
#pragma unroll
        for (int i = 0; i < 2; i++) dma.issue_one(ra, base, bad, st, wave_u, i);
        if constexpr (MX) {
            const __amdgpu_buffer_rsrc_t rw = make_rsrc(ws_base + (j < nk ? j : 0) * w_slab, (N - n0) * 64);
#pragma unroll
            for (int i = 0; i < 2; i++) dmaw.issue_one(rw, 0u, off, st + kOp, wave_u, i);
            const uint32_t blk = (uint32_t)j * 4u + 2u * ((uint32_t)wave_u & 1u) + ((uint32_t)lane >> 5);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, st + 2 * kOp + wave_u * 256, 4,
                                                     (int)((blk * (uint32_t)s_rows + s_row) | off), 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 2; i++) dma.issue_one(rb, base, bad, st + kOp, wave_u, i);
        }
    };
#pragma unroll
    for (int s = 0; s < S - 1; s++) issue(s, s);
    // Y_ref of this lane's outputs, in registers from the start: rows past M lie outside the resource and columns
    // past N get bit 31, both read as zero (and their accumulators are zero)
    const uint32_t N32 = (uint32_t)N;
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(MSE ? Yref + m0 * N : dY, MSE ? (M - m0) * N * 2 : 0);
    const __amdgpu_buffer_rsrc_t rd = make_rsrc(dY + m0 * N, (M - m0) * N * 2);
    uint32_t o_off[2];  // element (row wm 64 + 4 lh, column 32 j + lr of the wave's half); rows add N 2 bytes each
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const uint32_t col = (uint32_t)n0 + wn * 64 + j * 32 + lr;
        o_off[j] = (((uint32_t)(wm * 64 + 4 * lh) * N32 + col) * 2u) | (uint32_t)(col >= N32) << 31;
    }
    auto row_of = [](int i, int r) { return (uint32_t)(32 * i + 8 * (r / 4) + r % 4); };
    uint16_t y[2][2][16];
    if constexpr (MSE) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int r = 0; r < 16; r++)
                    y[i][j][r] = __builtin_amdgcn_raw_buffer_load_b16(ry, (int)(o_off[j] + row_of(i, r) * N32 * 2u), 0, 0);
    }
    f32x16_t acc[2][2];
    const f32x16_t zero = {};
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = zero;
    const uint32_t lds0 = lds_addr(smem);
    uint32_t a_off[2], b_off[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        a_off[h] = fwd_off(wm * 64 + lr, h * 2 + lh);
        b_off[h] = kOp + fwd_off(wn * 64 + lr, h * 2 + lh);
    }
    const uint32_t xs_off = 2 * kOp + lh * 128 + (uint32_t)(wm * 8 + (lr >> 2)) * 8u;
    const uint32_t ws_off = 2 * kOp + 512 + lh * 128 + (uint32_t)(wn * 8 + (lr >> 2)) * 8u;
    const uint32_t sc_b = (uint32_t)lr & 3u, sc_sel = sc_b | 0x0C00u | ((4u + sc_b) << 16) | 0x0C000000u;
    int sc = 0;
    for (int64_t kt = 0; kt < nk; kt++) {
        FOCUS_WAIT_VMCNT(kLoads * (S - 2));  // this thread's loads of slot kt have landed
        asm volatile("s_barrier" ::: "memory");
        const uint32_t st = lds0 + (uint32_t)sc * kStage;
        FwdStepFrags f;
        uint32_t sa[2], sb[2];
        if constexpr (MX) {
            read_step_mx(f, st + a_off[0], st + b_off[0], st + a_off[1], st + b_off[1], st + xs_off, st + ws_off);
#pragma unroll
            for (int i = 0; i < 2; i++) {
                sa[i] = __builtin_amdgcn_perm(f.x[1][i], f.x[0][i], sc_sel);
                sb[i] = __builtin_amdgcn_perm(f.w[1][i], f.w[0][i], sc_sel);
            }
        } else {
            read_step(f, st + a_off[0], st + b_off[0], st + a_off[1], st + b_off[1]);
        }
        // the stage that every wave was done with at the barrier; after the reads, which would queue behind the loads'
        // LDS writes (MXFP4: 5-9% faster)
        issue(kt + S - 1, sc == 0 ? S - 1 : sc - 1);
        static_for<2>([&](auto h) {
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    if constexpr (MX) {
                        typedef int v4i __attribute__((ext_vector_type(4)));
                        typedef int v8i __attribute__((ext_vector_type(8)));
                        const v4i a4 = __builtin_bit_cast(v4i, f.a[h][i]), b4 = __builtin_bit_cast(v4i, f.b[h][j]);
                        const v8i a8 = {a4[0], a4[1], a4[2], a4[3], 0, 0, 0, 0}, b8 = {b4[0], b4[1], b4[2], b4[3], 0, 0, 0, 0};
                        constexpr int ops = decltype(h)::value * 2;
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, acc[i][j], 4, 4, ops, (int)sa[i],
                                                                                    ops, (int)sb[j]);
                    } else {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[h][i], f.b[h][j], acc[i][j], 0, 0, 0);
                    }
                }
        });
        sc = sc == S - 1 ? 0 : sc + 1;
    }
    FOCUS_WAIT_VMCNT(0);  // the empty slots' zero writes must land before the LDS is handed on
    // D = Y_hat - Y_ref, dY = D dscale, column sums of D^2 (16 terms in fp32, then fp64, as with the large tiles)
    double csum[2] = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 2; i++) {
#pragma unroll
        for (int j = 0; j < 2; j++) {
            float sq = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                float o0 = acc[i][j][r], o1 = acc[i][j][r + 1];
                if constexpr (MSE) {
                    const float d0 = o0 - bf16_bits_to_f32(y[i][j][r]), d1 = o1 - bf16_bits_to_f32(y[i][j][r + 1]);
                    sq = __builtin_fmaf(d0, d0, sq);
                    sq = __builtin_fmaf(d1, d1, sq);
                    o0 = d0 * dscale;
                    o1 = d1 * dscale;
                }
                const uint32_t pk = cvt_pk_bf16(o0, o1);
                const uint32_t off = o_off[j] + row_of(i, r) * N32 * 2u;
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)pk, rd, (int)off, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(pk >> 16), rd, (int)(off + N32 * 2u), 0, 0);
            }
            csum[j] += (double)sq;
        }
    }
    if (!MSE) return;
#pragma unroll
    for (int j = 0; j < 2; j++) {
        csum[j] += __shfl_xor(csum[j], 32, 64);
        if (lh == 0) red[wm][wn * 64 + j * 32 + lr] = csum[j];
    }
    __syncthreads();
    if (t < kT && n0 + t < N) colpart[(int64_t)tm * N + n0 + t] = red[0][t] + red[1][t];
}

// ------------------------------------------------------------------------------------------------
// Backward (see bwd_mfma_kernel and bwd_mfma_mx_kernel): G^T = X_hat^T dY over one split's tokens, 32 per step,
// operands token-major in [32][128] bf16 tiles (256-byte rows, the 16-byte chunk index xor-ed with 4 (row % 4)).
constexpr int kRowB = kT * 2, kBOp = 32 * kRowB;  // 8 KB per operand and step

__device__ __forceinline__ uint32_t small_off(uint32_t r, uint32_t c) {
    return r * (uint32_t)kRowB + (((c >> 3) ^ ((r & 3u) << 2)) << 4) + (c & 7u) * 2u;
}

// Per-lane byte offset of the lower transposing read of the fragment at columns c (see ds_read_tr)
__device__ __forceinline__ uint32_t small_tr_off(uint32_t c, int lane) {
    const uint32_t j = lane & 15;
    return small_off(8 * (lane >> 5) + (j >> 2), c + 16 * ((lane >> 4) & 1) + 4 * (j & 3));
}

// A step's fragments, [half][32 columns]: 16 transposing reads and their wait in one block
struct BwdStepFrags {
    i16x4_t a[2][2][2], b[2][2][2];  // [half][columns][tokens + 0, + 4]
};
__device__ __forceinline__ void read_step_tr(BwdStepFrags &f, uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:1024\n\t"
        "ds_read_b64_tr_b16 %8, %18\n\tds_read_b64_tr_b16 %9, %18 offset:1024\n\t"
        "ds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:1024\n\t"
        "ds_read_b64_tr_b16 %10, %19\n\tds_read_b64_tr_b16 %11, %19 offset:1024\n\t"
        "ds_read_b64_tr_b16 %4, %16 offset:4096\n\tds_read_b64_tr_b16 %5, %16 offset:5120\n\t"
        "ds_read_b64_tr_b16 %12, %18 offset:4096\n\tds_read_b64_tr_b16 %13, %18 offset:5120\n\t"
        "ds_read_b64_tr_b16 %6, %17 offset:4096\n\tds_read_b64_tr_b16 %7, %17 offset:5120\n\t"
        "ds_read_b64_tr_b16 %14, %19 offset:4096\n\tds_read_b64_tr_b16 %15, %19 offset:5120\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(f.a[0][0][0]), "=&v"(f.a[0][0][1]), "=&v"(f.a[0][1][0]), "=&v"(f.a[0][1][1]), "=&v"(f.a[1][0][0]),
          "=&v"(f.a[1][0][1]), "=&v"(f.a[1][1][0]), "=&v"(f.a[1][1][1]), "=&v"(f.b[0][0][0]), "=&v"(f.b[0][0][1]),
          "=&v"(f.b[0][1][0]), "=&v"(f.b[0][1][1]), "=&v"(f.b[1][0][0]), "=&v"(f.b[1][0][1]), "=&v"(f.b[1][1][0]),
          "=&v"(f.b[1][1][1])
        : "v"(a0), "v"(a1), "v"(b0), "v"(b1)
        : "memory");
}

// A thread's 8 code bytes and scale byte, read and waited for in one block
__device__ __forceinline__ void read_codes(uint32_t codes, uint32_t scale, u32x2_t &w, uint32_t &sb) {
    asm volatile("ds_read_b64 %0, %2\n\tds_read_u8 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w), "=&v"(sb)
                 : "v"(codes), "v"(scale)
                 : "memory");
}

// With MX, X_hat is packed MXFP4 (Xc codes [M][K / 2], Xs bytes [K / 32][M]): a stage brings the dY tile, the codes
// ([32 tokens][64 bytes]) and the scale bytes ([4 blocks][32 tokens], one copy per wave), and a step before its use each
// thread converts 16 codes of the rows its own wave brought into one of two bf16 A stages. 2,048 x 1,024 x 2,560:
// bf16 26 us, packed 30 with the finishing kernel; on 256 x 256 tiles 39 and 40, most of it their epilogue.
template <int FMT, int WDT, bool MX>
__global__ void __launch_bounds__(kThreads, 2)
bwd_small_kernel(const uint16_t *__restrict__ dY, const void *__restrict__ X, const uint8_t *__restrict__ Xs, int64_t M,
                 int64_t N, int64_t K, int64_t chunk, const void *__restrict__ W, const float *__restrict__ s_fp,
                 const float *__restrict__ c, int sb_log2, const float *__restrict__ alpha_ptr, int ste_clip,
                 int e8m0_floor, float *__restrict__ part_s, float *__restrict__ part_c, int direct, uint32_t *flag,
                 int tiles_n) {
    constexpr int S = 4, kStep = 32;
    constexpr int kXOff = kBOp;                                   // X tile (or codes) after the dY tile
    constexpr int kScOff = kXOff + 32 * 64;                       // MX: the scale bytes, 256 bytes per wave
    constexpr int kStage = MX ? kScOff + 4 * 256 : 2 * kBOp;
    constexpr int kAOff = S * kStage;                             // MX: two bf16 stages of X
    constexpr int kLds = std::max(kAOff + (MX ? 2 * kBOp : 0), 64 * 1024);
    constexpr int kLoads = MX ? 5 : 4;
    __shared__ __attribute__((aligned(16))) char smem[kLds];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t id = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const uint32_t tile = id % gridDim.x;
    const int64_t k0 = (int64_t)(tile / (uint32_t)tiles_n) * kT, n0 = (int64_t)(tile % (uint32_t)tiles_n) * kT;
    const int64_t split = id / gridDim.x;
    const int64_t t_begin = split * chunk, t_end = std::min<int64_t>(M, t_begin + chunk);
    const int64_t nk = t_end > t_begin ? (t_end - t_begin + kStep - 1) / kStep : 0;
    lds_char *const lsm = (lds_char *)smem;
    // A 16-byte load instruction fills 4 token rows: lane L lands in row 4 q + L / 16, physical chunk L % 16 of block q;
    // a wave fills blocks 2 w and 2 w + 1. Columns past the matrix get bit 31; rows past the token range lie outside the
    // step's resource.
    auto tile_offs = [&](int64_t C, int64_t c0, uint32_t (&off)[2]) {
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const uint32_t row = 4u * (2u * wave_u + i) + ((uint32_t)lane >> 4);
            const uint32_t col = (uint32_t)c0 + (((uint32_t)lane & 15u) ^ ((row & 3u) << 2)) * 8u;
            off[i] = ((row * (uint32_t)C + col) * 2u) | (uint32_t)(col >= (uint32_t)C) << 31;
        }
    };
    uint32_t y_off[2], x_off[2];
    tile_offs(N, n0, y_off);
    if constexpr (!MX) tile_offs(K, k0, x_off);
    // MX: 4-byte loads; a wave fills code rows 8 w .. 8 w + 7 (four per instruction) and its own scale bytes (lanes 0-31:
    // block L / 8, tokens 4 (L % 8) .. + 3)
    const int64_t kc = K / 2;
    const uint32_t c_col = (uint32_t)(k0 / 2) + 4u * ((uint32_t)lane & 15u);
    const uint32_t c_bad = (uint32_t)(c_col >= (uint32_t)kc) << 31;
    const uint32_t s_blk = (uint32_t)(k0 / 32) + ((uint32_t)lane >> 3);
    const uint32_t s_off = s_blk * (uint32_t)M + 4u * ((uint32_t)lane & 7u);
    const uint32_t s_bad = (uint32_t)(lane >= 32 || s_blk >= (uint32_t)(K / 32)) << 31;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(Xs, MX ? (K / 32) * M : 0);
    auto issue = [&](int64_t j, int s) {
        const int64_t t0 = t_begin + j * kStep, rem = t_end - t0;
        const int64_t rows = rem <= 0 ? 0 : (rem < kStep ? rem : kStep), tb = rows ? t0 : 0;
        lds_char *const st = lsm + s * kStage;
        const __amdgpu_buffer_rsrc_t ry = make_rsrc(dY + tb * N, rows * N * 2);
        if constexpr (MX) {
            const __amdgpu_buffer_rsrc_t rc = make_rsrc(static_cast<const uint8_t *>(X) + tb * kc, rows * kc);
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const uint32_t blk = 2u * wave_u + i, row = 4u * blk + ((uint32_t)lane >> 4);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rc, st + kXOff + blk * 256, 4,
                                                         (int)((row * (uint32_t)kc + c_col) | c_bad), 0, 0, 0);
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, st + kScOff + wave_u * 256, 4,
                                                     (int)((s_off + (uint32_t)t0) | s_bad | (rows ? 0u : 0x80000000u)), 0, 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t rx = make_rsrc(static_cast<const uint16_t *>(X) + tb * K, rows * K * 2);
#pragma unroll
            for (int i = 0; i < 2; i++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, st + kXOff + (2 * wave_u + i) * 1024, 16, (int)x_off[i], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ry, st + (2 * wave_u + i) * 1024, 16, (int)y_off[i], 0, 0, 0);
    };
    const uint32_t lds0 = lds_addr(smem);
    // MX: this thread's codes 16 hb .. + 15 of token row, in the order of the rows that its wave brought
    const uint32_t row = (uint32_t)t >> 3, hb = (uint32_t)t & 7u;
    const uint32_t cv_dst0 = small_off(row, 16u * hb), cv_dst1 = small_off(row, 16u * hb + 8u);
    auto convert = [&](int s, int as) {
        u32x2_t w;
        uint32_t sb;
        const uint32_t st = lds0 + (uint32_t)s * kStage;
        read_codes(st + kXOff + row * 64u + 8u * hb, st + kScOff + (uint32_t)wave_u * 256u + 32u * (hb >> 1) + row, w, sb);
        const float scale = exp2i((int)sb - 127);
        u32x4_t v[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            v[h].x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w[h], scale, 0));
            v[h].y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w[h], scale, 1));
            v[h].z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w[h], scale, 2));
            v[h].w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w[h], scale, 3));
        }
        const uint32_t ab = lds0 + kAOff + (uint32_t)as * kBOp;
        asm volatile("ds_write_b128 %0, %1\n\tds_write_b128 %2, %3" : : "v"(ab + cv_dst0), "v"(v[0]), "v"(ab + cv_dst1), "v"(v[1]) : "memory");
    };
    uint32_t a_off[2], b_off[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        a_off[i] = small_tr_off(wm * 64 + i * 32, lane);
        b_off[i] = small_tr_off(wn * 64 + i * 32, lane);
    }
    f32x16_t acc[2][2];
    const f32x16_t zero = {};
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = zero;
#pragma unroll
    for (int s = 0; s < S - 1; s++) issue(s, s);
    if constexpr (MX) {
        FOCUS_WAIT_VMCNT(kLoads * (S - 2));  // this wave's own rows of slot 0
        asm volatile("" ::: "memory");
        convert(0, 0);
    }
    for (int64_t kt = 0; kt < nk; kt++) {
        const int sc = (int)(kt & (S - 1));
        // slot kt (MX: and kt + 1, whose codes are converted now) has landed here, and this thread's conversion of slot
        // kt is written; after the barrier everyone's, and every wave is done with step kt - 1's stages
        FOCUS_WAIT_VMCNT(kLoads * (MX ? S - 3 : S - 2));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const uint32_t st = lds0 + (uint32_t)sc * kStage;
        const uint32_t ab = MX ? lds0 + kAOff + (uint32_t)(kt & 1) * kBOp : st + kXOff;
        BwdStepFrags f;
        read_step_tr(f, ab + a_off[0], ab + a_off[1], st + b_off[0], st + b_off[1]);
        issue(kt + S - 1, (sc + S - 1) & (S - 1));
        static_for<2>([&](auto h) {
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    const i16x4_t va[2] = {f.a[h][i][0], f.a[h][i][1]}, vb[2] = {f.b[h][j][0], f.b[h][j][1]};
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, va),
                                                                        __builtin_bit_cast(bf16x8_t, vb), acc[i][j], 0, 0, 0);
                }
        });
        if constexpr (MX) convert((sc + 1) & (S - 1), (int)((kt + 1) & 1));
    }
    FOCUS_WAIT_VMCNT(0);  // the empty slots' zero writes must land before the LDS is used again
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    ste_epilogue<FMT, WDT, kT>(acc, k0, n0, split, N, K, W, s_fp, c, sb_log2, alpha_ptr, ste_clip, e8m0_floor, part_s,
                               part_c, direct, flag, smem);
}

}  // namespace

hipError_t launch_fwd_small(const void *X, const void *W, const void *Xs, const void *Ws, int64_t M, int64_t N, int64_t K,
                            const void *Yref, void *dY, float dscale, double *colpart, hipStream_t st) {
    const int tiles_n = (int)((N + kT - 1) / kT), tiles_m = (int)((M + kT - 1) / kT);
    const dim3 grid((unsigned)tiles_m * tiles_n);
    // Where the grid is at least twice as wide as high, groups of up to 8 row tiles are walked column by column, so that
    // a W panel is read by one XCD for them all; row after row, each row's XCDs read all of W (bf16 512 x 8,320 x 5,504:
    // 139 us, with 256 x 256 tiles 120, so 106). Narrower grids share enough either way, and square ones lost up to 8%.
    const bool wide = 2 * tiles_m <= tiles_n;
    const int groups = (tiles_m + 7) / 8, group = (tiles_m + groups - 1) / groups;
    const uint8_t *xs = static_cast<const uint8_t *>(Xs), *ws = static_cast<const uint8_t *>(Ws);
    const uint16_t *y = static_cast<const uint16_t *>(Yref);
    uint16_t *d = static_cast<uint16_t *>(dY);
#define FS(MSE, MX, WIDE) fwd_small_kernel<MSE, MX, WIDE><<<grid, kThreads, 0, st>>>(X, W, xs, ws, M, N, K, y, d, dscale, colpart, tiles_n, group)
#define FS_W(MSE, MX) if (!wide) FS(MSE, MX, false); else FS(MSE, MX, true)
    if (Xs) { if (Yref) { FS_W(true, true); } else { FS_W(false, true); } }
    else { if (Yref) { FS_W(true, false); } else { FS_W(false, false); } }
#undef FS_W
#undef FS
    return hipGetLastError();
}

hipError_t launch_bwd_small(int fmt, int w_dt, const void *dY, const void *X, const void *Xs, int64_t M, int64_t N, int64_t K,
                            int64_t chunk, int64_t splits, const void *W, const float *s_fp, const float *c, int sb,
                            const float *alpha, int ste_clip, int e8m0_floor, float *part_s, float *part_c, int direct,
                            uint32_t *flag, hipStream_t st) {
    const int tiles_k = (int)((K + kT - 1) / kT), tiles_n = (int)((N + kT - 1) / kT);
    int sbl = 0;
    while ((1 << sbl) < sb) sbl++;
    const dim3 grid((unsigned)tiles_k * tiles_n, (unsigned)splits);
    const uint16_t *dy = static_cast<const uint16_t *>(dY);
    const uint8_t *xs = static_cast<const uint8_t *>(Xs);
#define BS(F, WD, MX) bwd_small_kernel<F, WD, MX><<<grid, kThreads, 0, st>>>(dy, X, xs, M, N, K, chunk, W, s_fp, c, sbl, alpha, ste_clip, e8m0_floor, part_s, part_c, direct, flag, tiles_n)
    if (xs) { if (w_dt == kBF16) BS(kFmtMX, kBF16, true); else BS(kFmtMX, kF32, true); }
    else if (fmt == kFmtMX) { if (w_dt == kBF16) BS(kFmtMX, kBF16, false); else BS(kFmtMX, kF32, false); }
    else { if (w_dt == kBF16) BS(kFmtNV, kBF16, false); else BS(kFmtNV, kF32, false); }
#undef BS
    return hipGetLastError();
}

}  // namespace focus
