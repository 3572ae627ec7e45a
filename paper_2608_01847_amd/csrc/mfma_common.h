// Pieces shared by the bf16 / MXFP4 MFMA kernels of both tile sizes: tile order, operand staging with direct-to-LDS
// loads, transposing fragment reads and the straight-through epilogue.
#pragma once

#include "gemm_common.h"

namespace focus {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// Position t of a rows x cols tile grid in grouped order: groups of `group` row-tiles (default 4)
// are walked column by column, so the ~32 workgroups an XCD runs at once cover about 4 x 8 tiles and
// share 4 row panels and 8 column panels instead of 1 and 32.
constexpr uint32_t kGroupRows = 4;
__device__ __forceinline__ void grouped_tile(uint32_t t, uint32_t rows, uint32_t cols, uint32_t &r, uint32_t &c,
                                             uint32_t group = kGroupRows) {
    const uint32_t per_group = group * cols;
    const uint32_t first = (t / per_group) * group;
    const uint32_t in_group = rows - first < group ? rows - first : group;
    const uint32_t u = t % per_group;
    r = first + u % in_group;
    c = u / in_group;
}

// A direct-to-LDS load writes lane L's 16 bytes at LDS byte 16 L from the instruction's base, so
// each wave fills 1 KB blocks: lane L of block q lands in row 16 q + L / 4, physical chunk L % 4,
// which must hold logical chunk (L % 4) ^ fwd_key(row). The key depends on row bits 1-3 only,
// i.e. on L alone, so one step offset serves all of a wave's blocks. Offsets are in bytes of a row of
// `pitch` bytes (2 K for bf16 operands, K / 2 for packed FP4 codes); each thread's offsets at the
// first step are fixed for the whole tile.
template <int L = 4>  // loads per wave of a tile: 64 L rows
struct FwdDma {
    uint32_t lane_off[L];
    uint32_t cb;  // byte offset of this lane's chunk inside a step's 64 bytes of a row
    __device__ __forceinline__ void init(int64_t pitch, int wave, int lane) {
        cb = ((uint32_t)(lane & 3) ^ fwd_key((uint32_t)lane >> 2)) * 16u;
#pragma unroll
        for (int i = 0; i < L; i++) {
            const uint32_t row = (wave * L + i) * 16 + (lane >> 2);
            lane_off[i] = row * (uint32_t)pitch + cb;
        }
    }
    // Offset bits of the step whose row bytes start at b0: chunks at or past the row end get bit
    // 31 set, so they are out of range and read as zeros (an arithmetic mask, not a branch).
    __device__ __forceinline__ uint32_t step_bad(int64_t pitch, int64_t b0) const {
        const int32_t lim = (int32_t)(pitch - b0);
        return ((uint32_t)(lim - 1 - (int32_t)cb) >> 31) << 31;
    }
    // Load i (0..L - 1) of this wave for the step whose row bytes start at b0 = base.
    __device__ __forceinline__ void issue_one(__amdgpu_buffer_rsrc_t rs, uint32_t base, uint32_t bad,
                                              lds_char *dst, int wave, int i) const {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst + (wave * L + i) * 1024, 16,
                                                 (int)((lane_off[i] + base) | bad), 0, 0, 0);
    }
};

// Fragment of 32 operand rows (columns c .. c + 31 of a token-major tile) for the k16 step whose
// first token row is t0: lane l needs tokens t0 + 8 (l / 32) + 0..7 of column c + l % 32. A
// transposing read hands lane i of a 16-lane group element i % 4 of the 8-byte pieces addressed
// by lanes 4 e + i / 4 (e = 0..3); pointing lane j at row t0' + j / 4, columns c' + 4 (j % 4) .. + 3
// gives lane i tokens t0' .. t0' + 3 of column c' + i. Two reads (rows r and r + 4, the same
// swizzle) cover the 8 tokens.
//
// The reads are issued as inline assembly: the compiler's builtin for them carries no aliasing
// information, so the compiler would make every such read wait for all direct-to-LDS loads in
// flight (vmcnt(0)), draining the pipeline each step. The price is that the compiler does not
// track these reads: `tr_wait` must run before their registers are used, and it takes the
// fragments as operands so that no consumer can be scheduled above it.
typedef short i16x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lds_addr(const char *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

template <int OFF>
__device__ __forceinline__ i16x4_t ds_read_tr(uint32_t addr) {
    i16x4_t r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF));
    return r;
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

template <int OFF>
__device__ __forceinline__ u32x4_t ds_read_b128(uint32_t addr) {
    u32x4_t r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF));
    return r;
}

// Two fp32 values rounded to bf16 (to nearest, ties to even) in one instruction: lo in bits 0-15,
// hi in bits 16-31. Written out because the toolchain in use miscompiles the two-element vector
// conversion for gfx950 (it converts the first element only).
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
    return r;
}

// Fused straight-through epilogue of the backward kernels on G^T = acc (a TT k x TT n tile, TT = 256 or 128):
// per-split partial sums of G m w per sub-block and of G (q - m u) per block or, where the token range
// is not split (`direct`), the gradients themselves.
// acc[i][j][r] is G[n][k] for n = n0 + TT / 2 wn + 32 j + (lane % 32) and
// k = k0 + TT / 2 wm + 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4.
//
// Bound by vector instructions (TT = 256: one wave per SIMD, 256 elements per lane). G goes through LDS a quarter
// (accumulator column j, 64 rows n x 256 k, 64 KB, two buffers) at a time, or all at once (TT = 128, 64 KB), so that a thread then holds 8
// consecutive k of one row, as in the streaming fake-quant kernels: one scale, one coefficient and one
// division per 8 elements (u by div_by_scale where the whole wave's operands are in its range), 16-byte
// loads of W and 128-byte runs of c and of the sums, and the quarters run as a loop, whose code stays in
// the instruction cache. An epilogue in the accumulator layout (a lane holding 4 k of 32 rows, a true
// division per element, all 256 elements unrolled, 8- and 4-byte accesses 32 rows apart) made the whole
// backward of 2,048 x 1,024 x 2,560 (packed) take 65.4 us instead of 39.8, that of 3,001 x 1,368 x 2,128
// (NVFP4) 72.8 instead of 46.6 and that of 4,096 x 32,000 x 2,560 703 instead of 574.
template <int FMT, int WDT, int NCOEF, int TT>
__device__ __forceinline__ void ste_epilogue_n(const f32x16_t (&acc)[TT / 64][TT / 64], int64_t k0, int64_t n0, int64_t split,
                                               int64_t N, int64_t K, const void *__restrict__ W,
                                               const float *__restrict__ s_fp, const float *__restrict__ c, int sb_log2,
                                               const float *__restrict__ alpha_ptr, int ste_clip, int e8m0_floor,
                                               float *__restrict__ part_s, float *__restrict__ part_c, int direct,
                                               uint32_t *flag, char *smem) {
    constexpr int B = block_of(FMT);
    constexpr int WB = WDT == kBF16 ? 2 : 4;      // bytes per weight element
    constexpr int kItems = 8;                     // 8-element pieces per thread and quarter
    constexpr int kWords = WB * 8 / 16;           // 16-byte words of W per piece
    constexpr uint32_t kQuarters = TT == 256 ? 4u : 1u;
    constexpr uint32_t kQuarter = 64u * 1024u;
    constexpr uint32_t kLanes = TT / 8, kRows = 256 / kLanes;  // threads per row, rows per piece index
    constexpr uint32_t kPitch = TT * 4, kPeriod = 32 / kRows;  // bytes of a row; piece indexes per 32 rows
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lr = lane & 31, lh = lane >> 5;
    const float alpha = FMT == kFmtNV ? *alpha_ptr : 1.0f;
    const int64_t nb = K / B, ns = K >> sb_log2;
    const bool has_c = c != nullptr;
    bool bad = false;
    // W, S_fp and c of the tile's rows come through range-checked buffer loads: rows past N read as zeros,
    // and so do columns past K (bit 31 of the offset); both are kept out of the domain check, and their
    // sums are not stored (bit 31 again: the store is dropped). All offsets are 32-bit: a tile spans 256
    // rows of W (checked when the path is chosen), so none below bit 31 carries into or past it.
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(reinterpret_cast<const char *>(W) + n0 * K * WB, (N - n0) * K * WB);
    const __amdgpu_buffer_rsrc_t rsf = make_rsrc(s_fp + n0 * nb, (N - n0) * nb * 4);
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(has_c ? c + n0 * ns : s_fp, has_c ? (N - n0) * ns * 4 : 0);
    const __amdgpu_buffer_rsrc_t rps = make_rsrc(part_s + (split * N + n0) * nb, (N - n0) * nb * 4);
    const __amdgpu_buffer_rsrc_t rpc = make_rsrc(part_c + (split * N + n0) * ns, (N - n0) * ns * 4);
    const uint32_t K32 = (uint32_t)K, nb32 = (uint32_t)nb, ns32 = (uint32_t)ns;
    const uint32_t rows = N - n0 < TT ? (uint32_t)(N - n0) : (uint32_t)TT;
    // This thread's pieces of quarter q: k = kl .. kl + 7 of local rows r0 + kRows i (i = 0..7), which are rows
    // r0 + row_base(i, q) of the tile (TT = 256: local row rl is tile row 128 (rl / 32) + 32 q + rl % 32).
    const uint32_t kl = (uint32_t)k0 + 8u * ((uint32_t)t % kLanes), r0 = (uint32_t)t / kLanes;
    const bool k_ok = kl < K32;
    const uint32_t past = (uint32_t)!k_ok << 31;  // K < 2^31
    auto row_base = [](uint32_t i, uint32_t q) {
        return TT == 256 ? (i >> 2) * 128u + q * 32u + 8u * (i & 3u) : kRows * i;
    };
    const uint32_t w_off = (r0 * K32 * WB + kl * WB) | past, s_off = (r0 * nb32 + kl / B) * 4u | past,
                   c_off = (r0 * ns32 + (kl >> sb_log2)) * 4u | past;
    // stores of a sum over several threads are made by the first of them
    const uint32_t s_st = s_off | ((kl & (uint32_t)(B - 1)) ? 0x80000000u : 0u);
    const uint32_t c_st = c_off | (NCOEF == 1 && (kl & ((1u << sb_log2) - 1u)) ? 0x80000000u : 0u);
    u32x4 raw[kItems][kWords];
    float sv[kItems], cv[kItems][NCOEF];
    auto load_item = [&](auto i, uint32_t q) {
        const uint32_t rb = row_base(i, q);
#pragma unroll
        for (int h = 0; h < kWords; h++)
            raw[i][h] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(w_off + rb * K32 * WB + 16u * h), 0, 0);
        sv[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsf, (int)(s_off + rb * nb32 * 4u), 0, 0));
#pragma unroll
        for (int k = 0; k < NCOEF; k++)
            cv[i][k] = __uint_as_float(
                __builtin_amdgcn_raw_buffer_load_b32(rc, (int)(c_off + rb * ns32 * 4u + 4u * k), 0, 0));
    };
    static_for<kItems>([&](auto i) { load_item(i, 0u); });
    // 16-byte chunk ch (4 k) of local row rl lies at rl kPitch + 16 (ch ^ rl % 32): the xor spreads one chunk of
    // 32 rows (the writes) and the chunks of one row (the reads) over the banks
    const uint32_t wr = ((uint32_t)wn * (TT == 256 ? 32u : 64u) + lr) * kPitch +
                        (((uint32_t)wm * (TT / 8) + lh) ^ (uint32_t)lr) * 16u;
    uint32_t rd[kPeriod];  // chunk 2 (t % kLanes) of row r0 + kRows i, i < kPeriod; the next chunk is at rd ^ 16
#pragma unroll
    for (uint32_t i = 0; i < kPeriod; i++)
        rd[i] = (r0 + kRows * i) * kPitch + ((2u * ((uint32_t)t % kLanes)) ^ (r0 + kRows * i)) * 16u;
    __syncthreads();  // every wave is done with the operand stages
#pragma nounroll
    for (uint32_t q = 0; q < kQuarters; q++) {
        char *const buf = smem + (q & 1u) * kQuarter;
        auto put = [&](auto j) {
            static_for<TT / 16>([&](auto ig) {
                constexpr int i = ig / 4, g = ig % 4;
                const f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                *reinterpret_cast<f32x4 *>(buf + (wr ^ (16u * (8u * i + 2u * g))) + (TT == 256 ? 0u : 32u * kPitch * j)) = v;
            });
        };
        if constexpr (TT == 256) {
            if (q == 0u) put(std::integral_constant<int, 0>{});
            else if (q == 1u) put(std::integral_constant<int, 1>{});
            else if (q == 2u) put(std::integral_constant<int, 2>{});
            else put(std::integral_constant<int, 3>{});
        } else {
            static_for<TT / 64>(put);
        }
        // LDS only: the loads of W, s and c stay in flight. A buffer is written again two quarters later,
        // after the barrier that follows this quarter's reads.
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        f32x4 gv[2][2];  // G of this piece and of the next
        auto get = [&](auto i) {
            gv[i & 1][0] = *reinterpret_cast<const f32x4 *>(buf + rd[i % kPeriod] + (i / kPeriod) * 32u * kPitch);
            gv[i & 1][1] = *reinterpret_cast<const f32x4 *>(buf + (rd[i % kPeriod] ^ 16u) + (i / kPeriod) * 32u * kPitch);
        };
        get(std::integral_constant<int, 0>{});
        static_for<kItems>([&](auto i) {
            const uint32_t rb = row_base(i, q);
            const bool ok = k_ok && r0 + rb < rows;
            if constexpr (i + 1 < kItems) get(std::integral_constant<int, i + 1>{});
            float g[8], w[8];
#pragma unroll
            for (int e = 0; e < 8; e++) g[e] = gv[i & 1][e / 4][e % 4];
            bool fast;
            if constexpr (WDT == kBF16) {
                const uint4 p = make_uint4(raw[i][0].x, raw[i][0].y, raw[i][0].z, raw[i][0].w);
                fast = bf16x8_over_2p80(p) == 0u;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    w[2 * e] = __uint_as_float(raw[i][0][e] << 16);
                    w[2 * e + 1] = __uint_as_float(raw[i][0][e] & 0xFFFF0000u);
                }
            } else {
                uint32_t top = 0u;  // magnitudes as integers order like the values, NaN above all of them
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const uint32_t b = raw[i][e / 4][e % 4];
                    w[e] = __uint_as_float(b);
                    top = std::max(top, b & 0x7FFFFFFFu);
                }
                fast = top <= 0x67800000u;  // 2^80
            }
            uint32_t byte;
            bool nan = false;
            const float sdq = weight_sdq(FMT, sv[i], alpha, e8m0_floor, byte, nan);
            float cw[NCOEF];
#pragma unroll
            for (int k = 0; k < NCOEF; k++) {
                cw[k] = has_c ? cv[i][k] : 1.0f;
                nan = nan || bad_coeff(cw[k]);
            }
            bad = bad || (ok && nan);
            if (q + 1u < kQuarters) load_item(i, q + 1u);  // the next quarter's piece, into the registers just read
            // (a piece outside the tensor may divide by zero here; nothing of it is stored, and the other
            // pieces of its block lie outside too)
            float tc[NCOEF], ts;
            ste_piece<NCOEF>(g, w, sdq, cw, fast, ok, ste_clip, tc, ts);
            const uint32_t drop = ok ? 0u : 0x80000000u;
            if constexpr (NCOEF == 1) {
                if (sb_log2 >= 4) tc[0] += quad_xor<1>(tc[0]);
                if (sb_log2 >= 5) tc[0] += quad_xor<2>(tc[0]);
            }
#pragma unroll
            for (int k = 0; k < NCOEF; k++) {
                if (direct) tc[k] = -tc[k] / (cw[k] * cw[k]);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(tc[k]), rpc,
                                                      (int)((c_st + rb * ns32 * 4u + 4u * k) | drop), 0, 0);
            }
            ts += quad_xor<1>(ts);
            if (B == 32) ts += quad_xor<2>(ts);
            if (FMT == kFmtNV && direct) ts *= alpha;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ts), rps, (int)((s_st + rb * nb32 * 4u) | drop), 0, 0);
        });
    }
    if (bad) raise_domain_flag(flag);
}

template <int FMT, int WDT, int TT>
__device__ __forceinline__ void ste_epilogue(const f32x16_t (&acc)[TT / 64][TT / 64], int64_t k0, int64_t n0, int64_t split,
                                             int64_t N, int64_t K, const void *__restrict__ W,
                                             const float *__restrict__ s_fp, const float *__restrict__ c, int sb_log2,
                                             const float *__restrict__ alpha_ptr, int ste_clip, int e8m0_floor,
                                             float *__restrict__ part_s, float *__restrict__ part_c, int direct,
                                             uint32_t *flag, char *smem) {
    auto go = [&](auto nc) {
        ste_epilogue_n<FMT, WDT, decltype(nc)::value, TT>(acc, k0, n0, split, N, K, W, s_fp, c, sb_log2, alpha_ptr, ste_clip,
                                                      e8m0_floor, part_s, part_c, direct, flag, smem);
    };
    if (sb_log2 >= 3) go(std::integral_constant<int, 1>{});  // coefficients per 8 elements
    else if (sb_log2 == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
}

}  // namespace focus
