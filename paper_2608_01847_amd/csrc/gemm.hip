// Reconstruction GEMMs of the FOCUS step: planning, the LDS-tiled VALU kernels (shapes that the MFMA
// kernels do not take) with the fused MSE / straight-through epilogues, and the deterministic
// reductions that finish both. The bf16 and fp32 MFMA kernels live in gemm_mfma.hip and gemm_f32.hip.
#include "focus_device.h"
#include "gemm_common.h"
#include "internal.h"

namespace focus {

// ------------------------------------------------------------------------------------------------
// VALU forward: 64 x 64 output tile, 256 threads, 4 x 4 outputs per thread, K steps of 16.
// Epilogue: D = Y_hat - Y_ref, dY = D * dscale, per-column sums of D^2 over the tile's rows (fp64),
// written as colpart[mtile][n]. Plain mode (Yref == nullptr) stores Y_hat.
template <int DT>
__global__ void __launch_bounds__(256)
fwd_valu_kernel(const void *__restrict__ X, const void *__restrict__ W, int64_t M, int64_t N, int64_t K,
                const void *__restrict__ Yref, void *__restrict__ dY, float dscale,
                double *__restrict__ colpart) {
    __shared__ float As[16][68];
    __shared__ float Bs[16][68];
    __shared__ double cs[16][64];
    const int64_t m0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    float acc[4][4] = {};
    for (int64_t k0 = 0; k0 < K; k0 += 16) {
        for (int i = threadIdx.x; i < 64 * 16; i += 256) {
            const int r = i / 16, kk = i % 16;
            const int64_t gk = k0 + kk;
            const int64_t gm = m0 + r, gn = n0 + r;
            As[kk][r] = (gm < M && gk < K) ? load1(X, DT, gm * K + gk) : 0.0f;
            Bs[kk][r] = (gn < N && gk < K) ? load1(W, DT, gn * K + gk) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; kk++) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                a[i] = As[kk][ty * 4 + i];
                b[i] = Bs[kk][tx * 4 + i];
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 4; j++) acc[i][j] = __builtin_fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    double colsum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int64_t m = m0 + ty * 4 + i;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t n = n0 + tx * 4 + j;
            if (m < M && n < N) {
                const int64_t o = m * N + n;
                if (Yref) {
                    const float d = acc[i][j] - load1(Yref, DT, o);
                    store1(dY, DT, o, d * dscale);
                    colsum[j] += (double)d * (double)d;
                } else {
                    store1(dY, DT, o, acc[i][j]);
                }
            }
        }
    }
    if (!Yref) return;
#pragma unroll
    for (int j = 0; j < 4; j++) cs[ty][tx * 4 + j] = colsum[j];
    __syncthreads();
    if (threadIdx.x < 64 && n0 + threadIdx.x < N) {
        double s = 0.0;
        for (int r = 0; r < 16; r++) s += cs[r][threadIdx.x];
        colpart[(int64_t)blockIdx.y * N + n0 + threadIdx.x] = s;
    }
}

// ------------------------------------------------------------------------------------------------
// VALU backward: G tile of 64 (n) x 64 (k) reduced over the tokens [z*chunk, min(M,(z+1)*chunk)),
// then the fused straight-through epilogue (sums per sub-block and per block, see ste_terms).
template <int DT, int FMT, int WDT>
__global__ void __launch_bounds__(256)
bwd_valu_kernel(const void *__restrict__ dY, const void *__restrict__ X, int64_t M, int64_t N, int64_t K,
                int64_t chunk, const void *__restrict__ W, const float *__restrict__ s_fp,
                const float *__restrict__ c, int sb, const float *__restrict__ alpha_ptr, int ste_clip, int e8m0_floor,
                float *__restrict__ part_s, float *__restrict__ part_c, float *__restrict__ G_out,
                uint32_t *flag) {
    constexpr int B = block_of(FMT);
    __shared__ float As[16][68];
    __shared__ float Bs[16][68];
    __shared__ float Tc[64][65];
    __shared__ float Ts[64][65];
    const int64_t n0 = (int64_t)blockIdx.y * 64, kb = (int64_t)blockIdx.x * 64;
    const int64_t t0 = (int64_t)blockIdx.z * chunk, t1 = std::min<int64_t>(M, t0 + chunk);
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    float acc[4][4] = {};
    for (int64_t tb = t0; tb < t1; tb += 16) {
        for (int i = threadIdx.x; i < 64 * 16; i += 256) {
            const int r = i % 64, tt = i / 64;
            const int64_t t = tb + tt;
            As[tt][r] = (t < t1 && n0 + r < N) ? load1(dY, DT, t * N + n0 + r) : 0.0f;
            Bs[tt][r] = (t < t1 && kb + r < K) ? load1(X, DT, t * K + kb + r) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int tt = 0; tt < 16; tt++) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                a[i] = As[tt][ty * 4 + i];
                b[i] = Bs[tt][tx * 4 + i];
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 4; j++) acc[i][j] = __builtin_fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    const float alpha = FMT == kFmtNV ? *alpha_ptr : 1.0f;
    const int64_t nb = K / B, ns = K / sb;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int64_t n = n0 + ty * 4 + i;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t k = kb + tx * 4 + j;
            float tc = 0.0f, ts = 0.0f;
            if (n < N && k < K) {
                if (G_out) G_out[n * K + k] = acc[i][j];
                uint32_t byte;
                const float sdq = weight_sdq(FMT, s_fp[n * nb + k / B], alpha, e8m0_floor, byte, bad);
                const float cv = c ? c[n * ns + k / sb] : 1.0f;
                bad |= bad_coeff(cv);
                ste_terms(acc[i][j], load1(W, WDT, n * K + k), sdq, cv, ste_clip != 0, tc, ts);
            }
            Tc[ty * 4 + i][tx * 4 + j] = tc;
            Ts[ty * 4 + i][tx * 4 + j] = ts;
        }
    }
    __syncthreads();
    const int nsub = 64 / sb;
    for (int e = threadIdx.x; e < 64 * nsub; e += 256) {
        const int r = e / nsub, s = e % nsub;
        const int64_t n = n0 + r, k = kb + (int64_t)s * sb;
        if (n < N && k < K) {
            float sum = 0.0f;
            for (int x = 0; x < sb; x++) sum += Tc[r][s * sb + x];
            part_c[((int64_t)blockIdx.z * N + n) * ns + k / sb] = sum;
        }
    }
    constexpr int nblk = 64 / B;
    for (int e = threadIdx.x; e < 64 * nblk; e += 256) {
        const int r = e / nblk, s = e % nblk;
        const int64_t n = n0 + r, k = kb + (int64_t)s * B;
        if (n < N && k < K) {
            float sum = 0.0f;
            for (int x = 0; x < B; x++) sum += Ts[r][s * B + x];
            part_s[((int64_t)blockIdx.z * N + n) * nb + k / B] = sum;
        }
    }
    if (bad) raise_domain_flag(flag);
}

// ------------------------------------------------------------------------------------------------
// Deterministic finishing reductions (fixed summation order, no atomics).

// col_sq[n] = sum over m-tiles of colpart[mt][n] in a fixed order: 16 row groups (mt mod 16, each
// summed in ascending mt), then a fixed pairwise tree over the groups. A workgroup covers 16
// columns, so even a narrow layer spreads over many workgroups. Bound by the latency of its loads (each added before
// the next was issued): kAhead are in flight at a time, those past the end in bounds and left out.
// Partials of 256 x 9,728: 10.9 -> 8.2 us, of 256 x 2,560: 10.0 -> 4.8; the loss of 9,728 columns: 11.3 -> 4.6.
constexpr int kAhead = 8;
__global__ void __launch_bounds__(256)
colsum_kernel(const double *__restrict__ colpart, int64_t mtiles, int64_t N, double *__restrict__ col_sq) {
    __shared__ double red[16][16];
    const int cx = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int64_t n = (int64_t)blockIdx.x * 16 + cx;
    double s = 0.0;
    if (n < N)
        for (int64_t m0 = grp; m0 < mtiles; m0 += 16 * kAhead) {
            double v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; u++) v[u] = colpart[std::min<int64_t>(m0 + 16 * u, mtiles - 1) * N + n];
#pragma unroll
            for (int u = 0; u < kAhead; u++) s += m0 + 16 * u < mtiles ? v[u] : 0.0;
        }
    red[grp][cx] = s;
    __syncthreads();
    for (int w = 8; w > 0; w >>= 1) {
        if (grp < w) red[grp][cx] += red[grp + w][cx];
        __syncthreads();
    }
    if (grp == 0 && n < N) col_sq[n] = red[0][cx];
}

// loss = (sum over n of col_sq[n]) / (M N); one workgroup, strided partial sums then a fixed tree
__global__ void __launch_bounds__(256)
loss_kernel(const double *__restrict__ col_sq, int64_t N, double inv_mn, double *__restrict__ loss) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t n0 = threadIdx.x; n0 < N; n0 += 256 * kAhead) {
        double v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; u++) v[u] = col_sq[std::min<int64_t>(n0 + 256 * u, N - 1)];
#pragma unroll
        for (int u = 0; u < kAhead; u++) s += n0 + 256 * u < N ? v[u] : 0.0;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0] * inv_mn;
}

// Both of the above in one workgroup, where the partials are few (a launch costs more than their sums): a thread per
// column, the same order of additions. 4 x 256 partials take 3.9 us,
// where the two kernels take 4.4 and a launch more; at 16 x 1,024 (7.7) it is no longer ahead. At most 16 tile rows, one
// batch of loads: with a second batch behind it, 32 x 24 partials took 11.8 us, and 102 x 24 30, the two kernels 5.9.
constexpr int kFinishCols = 1024;
constexpr int64_t kFinishParts = 4096, kFinishRows = 16;
bool fwd_finish_in_one(int64_t mtiles, int64_t N) {
    return N <= kFinishCols && mtiles <= kFinishRows && mtiles * N <= kFinishParts;
}
__global__ void __launch_bounds__(1024)
fwd_finish_small_kernel(const double *__restrict__ colpart, int64_t mtiles, int64_t N, double *__restrict__ col_sq,
                        double inv_mn, double *__restrict__ loss) {
    __shared__ double cols[kFinishCols];
    __shared__ double part[256];
    for (int64_t n = threadIdx.x; n < N; n += 1024) {
        double s[16];
#pragma unroll
        for (int g = 0; g < 16; g++) s[g] = 0.0;
        for (int64_t m0 = 0; m0 < mtiles; m0 += 16) {
#pragma unroll
            for (int g = 0; g < 16; g++) {
                const int64_t mt = std::min<int64_t>(m0 + g, mtiles - 1);  // in bounds, left out past the last
                const double v = colpart[mt * N + n];
                s[g] += m0 + g < mtiles ? v : 0.0;
            }
        }
#pragma unroll
        for (int w = 8; w > 0; w >>= 1)
#pragma unroll
            for (int g = 0; g < w; g++) s[g] += s[g + w];
        col_sq[n] = cols[n] = s[0];
    }
    __syncthreads();
    if (!loss) return;
    double s = 0.0;
    if (threadIdx.x < 256) {
        for (int64_t n = threadIdx.x; n < N; n += 256) s += cols[n];
        part[threadIdx.x] = s;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = part[0] * inv_mn;
}

// grad_c = -(sum over splits of part_c) / c^2 ; grad_s = f * (sum over splits of part_s)
__global__ void __launch_bounds__(256)
bwd_finish_kernel(const float *__restrict__ part_s, const float *__restrict__ part_c, int64_t splits,
                  int64_t n_s, int64_t n_c, const float *__restrict__ c, const float *__restrict__ alpha_ptr,
                  int fmt, float *__restrict__ grad_s, float *__restrict__ grad_c) {
    const float f = fmt == kFmtNV ? *alpha_ptr : 1.0f;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_s + n_c; i += (int64_t)gridDim.x * 256) {
        if (i < n_c) {
            float s = 0.0f;
            for (int64_t z = 0; z < splits; z++) s += part_c[z * n_c + i];
            const float cv = c ? c[i] : 1.0f;
            grad_c[i] = -s / (cv * cv);
        } else {
            const int64_t j = i - n_c;
            float s = 0.0f;
            for (int64_t z = 0; z < splits; z++) s += part_s[z * n_s + j];
            grad_s[j] = fmt == kFmtNV ? s * f : s;
        }
    }
}

// ================================================================================================
// Planning and dispatch
// ================================================================================================

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Rows of a bf16 / MXFP4 forward tile: 128 x 128 tiles while they are at most two (MXFP4) or one and a half (bf16)
// per CU, else 256 x 256. With 264 small tiles (3,000 x 1,368 x 2,176) they took 22.3 and 40.6 us for 32.5 and 55.9,
// with 512 (2,048 x 4,096 x 4,096) 36.8 and 109 for 43.6 and 99, with 960 40 and 85 for 33 and 61.
int64_t fwd_tile_rows(int64_t M, int64_t N, bool mx) {
    return cdiv(M, kSmallTile) * cdiv(N, kSmallTile) <= (mx ? 2 * kMfmaConcurrentWgs : 3 * kMfmaConcurrentWgs / 2)
               ? kSmallTile : kMfmaTileM;
}

FwdPlan plan_fwd(int op_dt, int64_t M, int64_t N, int64_t K) {
    FwdPlan p;
    p.path = op_dt == kBF16 ? (mfma_fwd_supported(M, N, K) ? 1 : 0) : (f32_fwd_supported(M, N, K) ? 2 : 0);
    // fp32: 64 x 64 tiles where they give every CU one, else 32 x 32 with K split over the waves (128 x 256 x
    // 256 has 8 of the former and 32 of the latter)
    const bool small = p.path == 2 && cdiv(M, kF32Tile) * cdiv(N, kF32Tile) < kMfmaConcurrentWgs;
    p.tile_m = p.path == 1 ? fwd_tile_rows(M, N, false) : (small ? kF32Tile / 2 : 64);
    p.mtiles = cdiv(M, p.tile_m);
    p.ws_bytes = kWsHeader + (size_t)(p.mtiles * N + N) * sizeof(double);
    return p;
}

BwdPlan plan_bwd(int op_dt, int fmt, int sb, int64_t M, int64_t N, int64_t K, bool want_G) {
    BwdPlan p;
    p.path = op_dt == kBF16 ? (!want_G && mfma_bwd_supported(M, N, K) ? 1 : 0) : (f32_bwd_supported(M, N, K) ? 2 : 0);
    p.tile = p.path == 1 ? kMfmaTileN : 64;
    const int64_t step = p.path == 1 ? kMfmaTokenStep : (p.path == 2 ? kF32TokenStep : 16);
    const int64_t tiles = cdiv(N, p.tile) * cdiv(K, p.tile);
    const int64_t steps_total = cdiv(std::max<int64_t>(M, 1), step);
    const int64_t nb = K / block_of(fmt), ns = K / sb, sums = N * (nb + ns);  // sums of one split
    int64_t splits = 1;
    if (!want_G) {
        // The token range is split so that tiles * splits workgroups fill the chip in whole rounds (one 256 x 256
        // workgroup per CU on the MFMA path, several 64 x 64 ones on the VALU path): minimise the rounds, each the
        // steps of a split and an epilogue, and what splits cost beside them. Each split keeps >= 4 steps (fp32: 1).
        //  * MFMA path, in units of 0.02 us (190 layers of 512 to 131,072 tokens, each at up to 16 tilings and split
        //    counts): a 64-token step of a 256 x 256 tile 70, its epilogue 1040; more than one split a finishing
        //    launch (3 us) and its fp32 sums written and read once (3 TB/s). More splits have to promise 2% more than
        //    fewer, near ties went the other way (11,004 x 8,096 x 1,408: 241 us with one split, 263 with four).
        //  * fp32 path: a CU's matrix units are busy with one workgroup, so workgroups queue per CU too; its epilogue
        //    (64 x 64) costs about 3 of its 32-token steps (0.75 us each), the sums as above. Tiles that make 16
        //    rounds by themselves are not split (the last round is then a sixteenth of the time at most).
        // A cost is at least tiles * (steps_total * step + s * epilogue) / slots: past the best one the search ends.
        const int64_t slots = p.path == 0 ? 2048 : kMfmaConcurrentWgs;
        const int64_t step_cost = p.path == 1 ? 70 : 1, epilogue = p.path == 1 ? 1040 : (p.path == 2 ? 3 : 4);
        const int64_t launch = p.path == 1 ? 150 : 0, sums_rate = p.path == 1 ? 7500 : (p.path == 2 ? 281250 : 0);
        const int64_t margin = p.path == 1 ? 2 : 0;  // percent
        auto beside = [&](int64_t s) { return s > 1 && sums_rate ? launch + s * sums / sums_rate : 0; };
        const int64_t most = p.path == 2 ? (tiles >= 16 * slots ? 1 : steps_total) : steps_total / 4;
        const int64_t max_splits = std::max<int64_t>(1, std::min<int64_t>(most, 4096));
        int64_t best = -1;
        for (int64_t s = 1; s <= max_splits; s++) {
            if (best >= 0 && tiles * (step_cost * steps_total + s * epilogue) >= best * slots) break;
            const int64_t cost = cdiv(tiles * s, slots) * (step_cost * cdiv(steps_total, s) + epilogue) + beside(s);
            if (best < 0 || cost * (100 + margin) < best * 100) {
                best = cost;
                splits = s;
            }
        }
        // MFMA path: 128 x 128 tiles, two workgroups per CU, where the large tiles' epilogue would cost more than they
        // save (measured as above): a 64-token step takes 39 with one workgroup on the CU and 53 with two, their
        // epilogues 316 and 350; MXFP4, whose packed codes the small tiles convert twice as often, 48, 64, 330 and 280
        // (for its bf16 operands too, whose gradients have the packed ones' bits). (2,048 x 1,024 x 2,560: 26 to 30 us
        // for 39; 3,001 x 1,368 x 2,128: 39 for 47; 5,076 x 3,000 x 1,664: 79 to 95 for 71.)
        if (p.path == 1) {
            const int64_t small_tiles = cdiv(N, kSmallTile) * cdiv(K, kSmallTile);
            const bool mx = fmt == kFmtMX;
            const int64_t step1 = mx ? 48 : 39, ep1 = mx ? 330 : 316, step2 = mx ? 64 : 53, ep2 = mx ? 280 : 350;
            for (int64_t s = 1; s <= std::max<int64_t>(1, steps_total / 2) && small_tiles * s <= 8 * slots; s++) {
                if (small_tiles * (step2 * steps_total + s * ep2) >= best * 2 * slots) break;
                const int64_t per_cu = cdiv(small_tiles * s, slots), steps = cdiv(steps_total, s);
                const int64_t cost = per_cu / 2 * (step2 * steps + ep2) + per_cu % 2 * (step1 * steps + ep1) + beside(s);
                if (cost * (100 + margin) < best * 100) {
                    best = cost;
                    splits = s;
                    p.tile = kSmallTile;
                }
            }
        }
    }
    p.chunk = cdiv(steps_total, splits) * step;
    p.splits = std::max<int64_t>(1, cdiv(M, p.chunk));
    p.ws_bytes = kWsHeader + (size_t)(p.splits * sums) * sizeof(float);
    return p;
}

hipError_t launch_recon_fwd(const FwdPlan &p, int op_dt, const void *X, const void *W, int64_t M,
                            int64_t N, int64_t K, const void *Yref, void *dY, double *loss_out,
                            double *col_sq_opt, void *ws, hipStream_t st) {
    double *colpart = reinterpret_cast<double *>(reinterpret_cast<char *>(ws) + kWsHeader);
    double *col_sq = col_sq_opt ? col_sq_opt : colpart + p.mtiles * N;
    const float dscale = (float)(2.0 / ((double)M * (double)N));
    if (p.path == 1) {
        hipError_t e = p.tile_m == kSmallTile
                           ? launch_fwd_small(X, W, nullptr, nullptr, M, N, K, Yref, dY, dscale, colpart, st)
                           : launch_fwd_mfma(X, W, M, N, K, Yref, dY, dscale, colpart, st);
        if (e != hipSuccess) return e;
    } else if (p.path == 2) {
        hipError_t e = launch_fwd_f32((int)p.tile_m, static_cast<const float *>(X), static_cast<const float *>(W), M, N, K,
                                      static_cast<const float *>(Yref), static_cast<float *>(dY), dscale, colpart, st);
        if (e != hipSuccess) return e;
    } else {
        dim3 grid((unsigned)cdiv(N, 64), (unsigned)cdiv(M, 64));
        if (op_dt == kBF16) fwd_valu_kernel<kBF16><<<grid, 256, 0, st>>>(X, W, M, N, K, Yref, dY, dscale, colpart);
        else fwd_valu_kernel<kF32><<<grid, 256, 0, st>>>(X, W, M, N, K, Yref, dY, dscale, colpart);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!Yref) return hipSuccess;
    return launch_fwd_finish(p.mtiles, M, N, colpart, col_sq, loss_out, st);
}

// a split of the input gradient keeps >= 8 steps of 32 n
int64_t dx_max_splits(int64_t N) { return std::max<int64_t>(1, std::min<int64_t>(cdiv(N, 32) / 8, 64)); }

DxPlan plan_dx(int op_dt, int64_t M, int64_t N, int64_t K) {
    DxPlan p{0, 1, N, 0};
    if (op_dt != kBF16 || !mfma_dx_supported(M, N, K)) {  // (M and K are positive past this)
        p.ws_bytes = kWsHeader + ((size_t)N * (size_t)K * sizeof(float) + 255) / 256 * 256 + plan_fwd(op_dt, M, K, N).ws_bytes;
        return p;
    }
    p.path = 1;
    // Few output tiles leave CUs idle, so the n range is split to fill the chip in whole rounds: minimise
    // rounds * (32-n steps per split + 8 for the tile's end) plus the traffic of the splits' fp32 sums, written and
    // read once (about 4 MB in the time of a step); at most kDxSums, and none where the tiles already make four rounds.
    // (A quarter of kDxSums, one round of tiles, took up to a quarter longer by this measure: 5,779 x 13,728 x 1,344.)
    const int64_t tiles = cdiv(M, kMfmaTileM) * cdiv(K, kMfmaTileK), steps = cdiv(std::max<int64_t>(N, 1), 32);
    int64_t best = -1;
    const int64_t most = tiles >= 4 * kMfmaConcurrentWgs
                             ? 1
                             : std::min<int64_t>(dx_max_splits(N), kDxSums / (M * K));
    for (int64_t s = 1; s <= std::max<int64_t>(1, most); s++) {
        const int64_t cost = cdiv(tiles * s, kMfmaConcurrentWgs) * (cdiv(steps, s) + 8) +
                             (s > 1 ? s * M * K * 8 / 4000000 + 4 : 0);
        if (best < 0 || cost < best) best = cost, p.splits = s;
    }
    p.chunk = cdiv(steps, p.splits) * 32;
    p.splits = std::max<int64_t>(1, cdiv(N, p.chunk));
    p.ws_bytes = kWsHeader + (p.splits > 1 ? (size_t)(p.splits * M * K) * sizeof(float) : 0);
    return p;
}

hipError_t launch_recon_dx(const DxPlan &p, int op_dt, const void *dY, const void *W_hat, int64_t M, int64_t N, int64_t K,
                           void *dX, void *ws, hipStream_t st) {
    char *const base = static_cast<char *>(ws) + kWsHeader;
    if (p.path == 1)
        return launch_dx_mfma(dY, W_hat, M, N, K, p.chunk, p.splits, dX, reinterpret_cast<float *>(base), st);
    hipError_t e = launch_transpose(op_dt, W_hat, N, K, base, st);
    if (e != hipSuccess) return e;
    // dX_hat [M][K] = dY [M][N] (W_hat^T [K][N])^T: the forward GEMM's plain product with N as the contraction
    return launch_recon_fwd(plan_fwd(op_dt, M, K, N), op_dt, dY, base, M, K, N, nullptr, dX, nullptr, nullptr,
                            base + ((size_t)N * (size_t)K * sizeof(float) + 255) / 256 * 256, st);
}

hipError_t launch_fwd_finish(int64_t mtiles, int64_t M, int64_t N, const double *colpart, double *col_sq,
                             double *loss_out, hipStream_t st) {
    if (fwd_finish_in_one(mtiles, N)) {
        fwd_finish_small_kernel<<<1, 1024, 0, st>>>(colpart, mtiles, N, col_sq, 1.0 / ((double)M * (double)N), loss_out);
        return hipGetLastError();
    }
    colsum_kernel<<<(unsigned)cdiv(N, 16), 256, 0, st>>>(colpart, mtiles, N, col_sq);
    if (loss_out) loss_kernel<<<1, 256, 0, st>>>(col_sq, N, 1.0 / ((double)M * (double)N), loss_out);
    return hipGetLastError();
}

hipError_t launch_recon_fwd_mx(const void *Xc, const void *Xs, const void *Wc, const void *Ws, int64_t M, int64_t N,
                               int64_t K, const void *Yref, void *dY, double *loss_out, double *col_sq_opt, void *ws,
                               hipStream_t st) {
    const int64_t rows = fwd_tile_rows(M, N, true), mtiles = cdiv(M, rows);
    double *colpart = reinterpret_cast<double *>(reinterpret_cast<char *>(ws) + kWsHeader);
    double *col_sq = col_sq_opt ? col_sq_opt : colpart + mtiles * N;
    const float dscale = (float)(2.0 / ((double)M * (double)N));
    hipError_t e = rows == kSmallTile ? launch_fwd_small(Xc, Wc, Xs, Ws, M, N, K, Yref, dY, dscale, colpart, st)
                                      : launch_fwd_mfma_mx(Xc, Xs, Wc, Ws, M, N, K, Yref, dY, dscale, colpart, st);
    if (e != hipSuccess || !Yref) return e;
    return launch_fwd_finish(mtiles, M, N, colpart, col_sq, loss_out, st);
}

hipError_t launch_recon_bwd(const BwdPlan &p, int op_dt, int fmt, int sb, int ste_clip, int e8m0_floor, const void *dY,
                            const void *X, int64_t M, int64_t N, int64_t K, const void *W, int w_dt,
                            const float *s_fp, const float *c, const float *alpha, float *grad_s,
                            float *grad_c, float *G_out, void *ws, uint32_t *flag, hipStream_t st) {
    const int64_t nb = K / block_of(fmt), ns = K / sb;
    float *part_s = reinterpret_cast<float *>(reinterpret_cast<char *>(ws) + kWsHeader);
    float *part_c = part_s + p.splits * N * nb;
    if (p.path == 1) {
        // one split: the kernel writes the gradients, nothing is left to sum
        const int direct = p.splits == 1;
        float *const gs = direct ? grad_s : part_s, *const gc = direct ? grad_c : part_c;
        hipError_t e = p.tile == kSmallTile
                           ? launch_bwd_small(fmt, w_dt, dY, X, nullptr, M, N, K, p.chunk, p.splits, W, s_fp, c, sb, alpha,
                                              ste_clip, e8m0_floor, gs, gc, direct, flag, st)
                           : launch_bwd_mfma(fmt, w_dt, dY, X, M, N, K, p.chunk, p.splits, W, s_fp, c, sb, alpha, ste_clip,
                                             e8m0_floor, gs, gc, direct, flag, st);
        if (e != hipSuccess || direct) return e;
    } else if (p.path == 2) {
        const int direct = p.splits == 1;
        hipError_t e = launch_bwd_f32(fmt, w_dt, static_cast<const float *>(dY), static_cast<const float *>(X), M, N, K,
                                      p.chunk, p.splits, W, s_fp, c, sb, alpha, ste_clip, e8m0_floor,
                                      direct ? grad_s : part_s, direct ? grad_c : part_c, direct, G_out, flag, st);
        if (e != hipSuccess || direct) return e;
    } else {
        dim3 grid((unsigned)cdiv(K, 64), (unsigned)cdiv(N, 64), (unsigned)p.splits);
#define BV(D, F, WD) bwd_valu_kernel<D, F, WD><<<grid, 256, 0, st>>>(dY, X, M, N, K, p.chunk, W, s_fp, c, sb, alpha, ste_clip, e8m0_floor, part_s, part_c, G_out, flag)
        if (op_dt == kBF16) {
            if (fmt == kFmtMX) { if (w_dt == kBF16) BV(kBF16, kFmtMX, kBF16); else BV(kBF16, kFmtMX, kF32); }
            else { if (w_dt == kBF16) BV(kBF16, kFmtNV, kBF16); else BV(kBF16, kFmtNV, kF32); }
        } else {
            if (fmt == kFmtMX) { if (w_dt == kBF16) BV(kF32, kFmtMX, kBF16); else BV(kF32, kFmtMX, kF32); }
            else { if (w_dt == kBF16) BV(kF32, kFmtNV, kBF16); else BV(kF32, kFmtNV, kF32); }
        }
#undef BV
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int64_t total = N * (nb + ns);
    const unsigned g = (unsigned)std::min<int64_t>(std::max<int64_t>(cdiv(total, 256), 1), kStreamGridCap);
    bwd_finish_kernel<<<g, 256, 0, st>>>(part_s, part_c, p.splits, N * nb, N * ns, c, alpha, fmt, grad_s, grad_c);
    return hipGetLastError();
}

hipError_t launch_recon_bwd_mx(const BwdPlan &p, int sb, int ste_clip, int e8m0_floor, const void *dY, const void *Xc,
                               const void *Xs, int64_t M, int64_t N, int64_t K, const void *W, int w_dt,
                               const float *s_fp, const float *c, float *grad_s, float *grad_c, void *ws,
                               uint32_t *flag, hipStream_t st) {
    const int64_t nb = K / 32, ns = K / sb;
    float *part_s = reinterpret_cast<float *>(reinterpret_cast<char *>(ws) + kWsHeader);
    float *part_c = part_s + p.splits * N * nb;
    const int direct = p.splits == 1;  // the kernel writes the gradients, nothing is left to sum
    float *const gs = direct ? grad_s : part_s, *const gc = direct ? grad_c : part_c;
    hipError_t e = p.tile == kSmallTile
                       ? launch_bwd_small(kFmtMX, w_dt, dY, Xc, Xs, M, N, K, p.chunk, p.splits, W, s_fp, c, sb, nullptr,
                                          ste_clip, e8m0_floor, gs, gc, direct, flag, st)
                       : launch_bwd_mfma_mx(w_dt, dY, Xc, Xs, M, N, K, p.chunk, p.splits, W, s_fp, c, sb, ste_clip,
                                            e8m0_floor, gs, gc, direct, flag, st);
    if (e != hipSuccess || direct) return e;
    const int64_t total = N * (nb + ns);
    const unsigned g = (unsigned)std::min<int64_t>(std::max<int64_t>(cdiv(total, 256), 1), kStreamGridCap);
    bwd_finish_kernel<<<g, 256, 0, st>>>(part_s, part_c, p.splits, N * nb, N * ns, c, nullptr, kFmtMX, grad_s, grad_c);
    return hipGetLastError();
}

}  // namespace focus
