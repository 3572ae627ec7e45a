// Pieces shared by the bf16 / MXFP4 MFMA kernels of both tile sizes: operand staging with direct-to-LDS loads
// and transposing fragment reads.
#pragma once

#include "gemm_common.h"

namespace focus {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

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

}  // namespace focus
