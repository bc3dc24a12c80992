// What the two attention kernels (attn.hip, attn_split.hip) share: constants of the softmax and lane operations.
#pragma once
#include "common.hpp"

namespace sparge {

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr int MAGIC_I = 0x4B400000;      // bit pattern of 12582912.0f = 1.5 * 2^23
constexpr float MAGIC_F = 12582912.0f;
// log2 units: P~ <= 2^8 (16-bit P~V) or 2^2 (FP8 P~V) relative to the reference maximum
static_assert(SPARGE_REF_SLACK_LOG2 == 8 && SPARGE_REF_SLACK_LOG2_FP8 == 2,
              "gen_attn_loop.py encodes the same thresholds (RESCALE_T)");
constexpr int PV_FP8 = 2;  // third kind of P~V product next to SPARGE_F16 / SPARGE_BF16

// 32x32x16 MFMA on 16-bit operands given as raw register quads.
template <int DT>
__device__ __forceinline__ v16f mfma16(v4i a, v4i b, v16f c) {
    if constexpr (DT == SPARGE_BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
}

// The value held by the lane 32 positions away, combined with the own one (v_permlane32_swap).
__device__ __forceinline__ float max_across_halves(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_across_halves(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float uniform(float v) {  // a wave-uniform float, moved to a scalar register
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}

// 16-byte global -> LDS copy that bypasses registers (LDS-DMA): lane L copies 16 bytes from
// gbase + lane_offset to lds_base + 16 L (lds_base wave-uniform).  Issued through inline assembly on
// purpose: the compiler then does not order later LDS reads behind the copy; the kernel waits for
// its copies itself (dma_wait) right before the barrier that publishes the tile.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)(p)));
}
// (to lds_base + the constant step: one scalar register serves a run of copies)
__device__ __forceinline__ void dma16_at(const void* gbase /*wave-uniform*/, uint32_t lane_offset, uint32_t lds_base, int step) {
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_offset), "s"(gbase), "s"(lds_base), "n"(step)
                 : "memory", "scc");
}
__device__ __forceinline__ void dma16(const void* gbase /*wave-uniform*/, uint32_t lane_offset, const void* lds_base) {
    dma16_at(gbase, lane_offset, lds_address(lds_base), 0);
}
// Wait until at most N of this wave's copies (the N most recent ones) are still in flight.
template <int N>
__device__ __forceinline__ void dma_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// LDS tiles are unpadded; bank conflicts of the 16-byte operand reads are avoided by XOR-ing the
// 16-byte chunk index of a row with a few row bits (applied on the global side of the copy).
template <int ROW_BYTES>
__device__ __forceinline__ int swz(int row) {
    return ROW_BYTES == 256 ? (row & 15) : ROW_BYTES == 128 ? ((row >> 1) & 7) : ((row >> 2) & 3);
}

}  // namespace

}  // namespace sparge
