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
template <bool MSE, bool MX>
__global__ void __launch_bounds__(kThreads, 2)
fwd_small_kernel(const void *__restrict__ X, const void *__restrict__ W, const uint8_t *__restrict__ Xs,
                 const uint8_t *__restrict__ Ws, int64_t M, int64_t N, int64_t K, const uint16_t *__restrict__ Yref,
                 uint16_t *__restrict__ dY, float dscale, double *__restrict__ colpart, int tiles_n) {
    constexpr int S = 4, kOp = kT * 64, kStage = 2 * kOp + (MX ? 1024 : 0);
    constexpr int kLoads = MX ? 5 : 4;     // loads per slot per thread
    constexpr int kKStep = MX ? 128 : 32;  // k per step
    __shared__ __attribute__((aligned(16))) char smem[S * kStage];
    __shared__ double red[2][kT];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31, lh = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const uint32_t tm = tile / (uint32_t)tiles_n, tn = tile % (uint32_t)tiles_n;
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

}  // namespace

hipError_t launch_fwd_small(const void *X, const void *W, const void *Xs, const void *Ws, int64_t M, int64_t N, int64_t K,
                            const void *Yref, void *dY, float dscale, double *colpart, hipStream_t st) {
    const int tiles_n = (int)((N + kT - 1) / kT);
    const dim3 grid((unsigned)((M + kT - 1) / kT) * tiles_n);
    const uint8_t *xs = static_cast<const uint8_t *>(Xs), *ws = static_cast<const uint8_t *>(Ws);
    const uint16_t *y = static_cast<const uint16_t *>(Yref);
    uint16_t *d = static_cast<uint16_t *>(dY);
#define FS(MSE, MX) fwd_small_kernel<MSE, MX><<<grid, kThreads, 0, st>>>(X, W, xs, ws, M, N, K, y, d, dscale, colpart, tiles_n)
    if (Xs) { if (Yref) FS(true, true); else FS(false, true); }
    else { if (Yref) FS(true, false); else FS(false, false); }
#undef FS
    return hipGetLastError();
}

}  // namespace focus
