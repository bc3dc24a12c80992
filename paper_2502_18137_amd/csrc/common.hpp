// Internal declarations shared by the HIP translation units of libsparge (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "sparge.h"

namespace sparge {

constexpr int BQ = SPARGE_BQ;         // query rows per block (Alg. 1 line 2; App. A.1)
constexpr int BK = SPARGE_BK;         // key rows per block
constexpr int RG = SPARGE_ROW_GROUP;  // rows per stage-2 row group (b_q / c_w)

// (batch, head) pair whose operands pair bh uses; index of its per-head parameters, `own`: pair behind the dense ones.  The
// divisions stay behind branches that an ordinary call never takes.
__host__ __device__ inline int operand_of(int bh, int op_bh) {
    if (bh < op_bh) return bh;
    asm volatile("");
    return bh % op_bh;
}
__host__ __device__ inline int param_of(int own, int h, int by_setting, int op_bh) {
    if (!by_setting) return h;
    asm volatile("");
    return own / op_bh;
}
struct Shape {
    int B, H, N, d, dtype;
    long long sb, sh, sn;  // element strides of the 16-bit tensors
    int Tm, Tn;
    int pv_fp8;            // P~V product in FP8 (E4M3) instead of the tensors' 16-bit type
    int qk16;              // Q K^T product on the 16-bit tensors themselves instead of their INT8 quantization
    // Several settings of the same operands in one launch (the hyper-parameter search): (batch, head) pairs beyond op_bh
    // use the operands of those before them, pair by pair.  The first dense_bh pairs keep every block and count nothing;
    // mask and counters begin behind them.
    int op_bh;             // (batch, head) pairs that have operands of their own; an ordinary call: B H
    int dense_bh;
    int by_setting;        // the per-head parameters (tau, theta, lambda) are one value per setting instead
    int one_mask;          // the mask has op_bh pairs: one for all settings

    __host__ __device__ int operand(int bh) const { return operand_of(bh, op_bh); }
    __host__ __device__ int param(int own, int h) const { return param_of(own, h, by_setting, op_bh); }
};

// Per-head scalars travel to the device inside the kernel argument block.
struct HeadParams {
    float v[SPARGE_MAX_HEADS];
};

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v8f __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// The value another lane of the same row of 16 holds, through a DPP move (vector ALU, no LDS traffic).
//   PARTNER 1, 2, 8: the value of lane ^ PARTNER (quad permutes, rotation by 8 inside a row of 16).
//   PARTNER 4: the value of lane ^ 4 (two shifts by 4, each written to the banks it is right for).
//   PARTNER 7, 15: the value of lane 7 - lane % 8 of the same group of 8, of lane 15 - lane % 16 of the same
//   row (mirrors, one instruction).  They serve as ^4 (^8) ONLY where the lanes of each group of 4 (of 8)
//   already hold the same value.
template <int PARTNER>
__device__ __forceinline__ uint32_t row_xchg(uint32_t v) {
    static_assert(PARTNER == 1 || PARTNER == 2 || PARTNER == 4 || PARTNER == 8 || PARTNER == 7 || PARTNER == 15,
                  "no such exchange");
    if constexpr (PARTNER == 4) {
        // row_shl:4 brings lane + 4 (banks 0 and 2 take it), row_shr:4 brings lane - 4 (banks 1 and 3)
        const int up = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x104, 0xF, 0x5, false);
        return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(up, static_cast<int>(v), 0x114, 0xF, 0xA, false));
    } else {
        constexpr int CTRL = PARTNER == 1 ? 0xB1 : PARTNER == 2 ? 0x4E : PARTNER == 7 ? 0x141 : PARTNER == 15 ? 0x140 : 0x128;
        // every lane has a source inside its row; bound_ctrl tells the compiler that the destination's old
        // value is never kept, which saves a register preload and its wait states per exchange
        return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, true));
    }
}

// 16-bit storage -> fp32 (exact).  DT: SPARGE_F16 or SPARGE_BF16.
template <int DT>
__device__ __forceinline__ float cvt16(uint16_t bits) {
    if constexpr (DT == SPARGE_BF16) {
        return __uint_as_float(static_cast<uint32_t>(bits) << 16);
    } else {
        _Float16 h;
        __builtin_memcpy(&h, &bits, 2);
        return static_cast<float>(h);
    }
}

// fp32 -> 16-bit storage, round to nearest even.
template <int DT>
__device__ __forceinline__ uint16_t cvt_to16(float f) {
    uint16_t bits;
    if constexpr (DT == SPARGE_BF16) {
        __bf16 h = static_cast<__bf16>(f);
        __builtin_memcpy(&bits, &h, 2);
    } else {
        _Float16 h = static_cast<_Float16>(f);
        __builtin_memcpy(&bits, &h, 2);
    }
    return bits;
}

// Order of the attention kernel's work items.  Items are numbered g = (b H + h) T_m + q; q counts a head's Q
// blocks from the last one down when the attention is causal (i = T_m - 1 - q: longest rows first), up
// otherwise (i = q).  They are cut into 8 contiguous ranges of `per_range` items, one per XCD, and a range hands
// out its items through a counter: p = 0, 1, ... -> the item returned here, for the range that starts at r0 and
// holds len items.  Non-causal: in index order.  Causal: in two passes over the range's heads, first the longer
// half of every head's rows (q < T_m - T_m / 2), head by head, then the shorter halves -- so that the items a
// range ends with are short whichever head they belong to (with whole heads one after the other the long rows
// of the last head start late and a tenth of the slot time at the causal language shape was an idle tail).
__host__ __device__ inline int range_item(int r0, int len, int p, int Tm, bool causal) {
    if (!causal) return r0 + p;
    const int r1 = r0 + len, longer = Tm - Tm / 2;
    const int h0 = r0 / Tm, h1 = (r1 - 1) / Tm;
    for (int pass = 0; pass < 2; ++pass) {
        const int lo = pass ? longer : 0, hi = pass ? Tm : longer;  // the q of this pass inside a head
        // the range's first head (it may begin inside it), the whole heads after it, its last head
        const int a0 = r0 - h0 * Tm > lo ? r0 - h0 * Tm : lo;
        const int b0 = r1 - h0 * Tm < hi ? r1 - h0 * Tm : hi;
        const int c0 = b0 > a0 ? b0 - a0 : 0;
        if (p < c0) return h0 * Tm + a0 + p;
        p -= c0;
        if (h1 > h0) {
            const int whole = (h1 - h0 - 1) * (hi - lo);
            if (p < whole) return (h0 + 1 + p / (hi - lo)) * Tm + lo + p % (hi - lo);
            p -= whole;
            const int b1 = r1 - h1 * Tm < hi ? r1 - h1 * Tm : hi;
            const int c1 = b1 > lo ? b1 - lo : 0;
            if (p < c1) return h1 * Tm + lo + p;
            p -= c1;
        }
    }
    return -1;  // p >= len
}

// What has to be set before an attention launch, by whatever kernel of the call runs earlier (a kernel of its own
// costs 5 us of a call): the item counters of its work distribution, one per XCD range, 128 bytes apart, to `start`
// (the items of each range that the launch's workgroups take without asking; counters null: every item has a
// workgroup of its own), and the caller's n_stats execution counters to zero (stats null: none).
constexpr int QUEUE_PITCH = 32;
constexpr size_t ATTN_QUEUE_BYTES = 1024;
static_assert(8 * QUEUE_PITCH * sizeof(unsigned int) == ATTN_QUEUE_BYTES, "eight counters, 128 bytes apart");
struct AttnStart {
    unsigned int* counters;
    unsigned int start;
    int n_stats;
    unsigned long long* stats;
};
// (called by all threads of each of `parts` workgroups of 256.  One is enough inside the block statistics, which hide
// it; a launch of its own takes one per 256 execution counters: 1028 against 1063 us for sparge_attn_quantized on
// 65408 heads)
__device__ __forceinline__ void set_start(const AttnStart& a, int part, int parts) {
    if (a.counters && part == 0 && threadIdx.x < 8) a.counters[threadIdx.x * QUEUE_PITCH] = a.start;
    if (a.stats)
        for (int n = part * 256 + static_cast<int>(threadIdx.x); n < a.n_stats; n += parts * 256) a.stats[n] = 0ull;
}

// ---- kernel launchers (host functions defined next to their kernels) ----------------------------
// Block statistics of Q and K: pooled means of Q (+ its INT8 quantization if Qq), per-block channel sums of K (transposed
// [B,H,d,Tn]), self-similarities; and what `start` asks for.  sim_q null: only
// what the quantization of Q and the mean of K need (Qq, q_scale, ksum_t).
hipError_t launch_block_stats(const void* Q, const void* K, const Shape& s, double* pooled_q, double* ksum_t,
                              double* sim_q, double* sim_k, int8_t* Qq, float* q_scale, AttnStart start, hipStream_t st);
// Short calls take the block statistics (and V tiles) in one launch and the predictor with the K quantization in
// another.  Up to 256 key blocks (a row's logits fit the LDS of a workgroup of 8 rows at full occupancy) and as many
// elements per tensor as below: a launch, an event and a wait saved are then worth more than what the passes lose in one
// kernel (the registers of the hungriest, the mean summed once per workgroup).  Separate launches against these, us, whole
// forward pass and predictor alone: 81 / 22, 24 / 18 at 4 x 64 x 64; 172 / 166, 37.4 / 31.4 at 192 x 1024 x 128;
// 324 / 317, 35.1 / 32.6 at 16 x 8192 x 128; 468 / 471, 41.6 / 40.2 at 24 x 8192 x 128 (on the line); 373 / 356,
// 27.4 / 24.9 at 8, 531 / 519, 32.6 / 28.7 at 12 and 694 / 677, 36.0 / 32.5 at 16 x 16384 x 64 (on the line);
// 564 / 558, 37.2 / 37.3 at 8 x 16384 x 128 (on the line).  Beyond it the two part: 851 / 841, 40.8 / 42.9 at
// 20 x 16384 x 64, 819 / 830, 44.4 / 44.2 at 12 x 16384 x 128, 490 / 487, 40.2 / 37.6 at 12 x 12000 x 128.
inline bool short_call(const Shape& s) {
    return s.Tn <= 256 && (long long)s.B * s.H * s.N * s.d <= (s.Tn <= 128 ? 3ll << 23 : 1ll << 24);
}
// Short calls: all of launch_block_stats in one launch, with V re-tiled as launch_v_tiles does if v_tiles.
hipError_t launch_prep(const void* Q, const void* K, const void* V, const Shape& s, double* pooled_q, double* ksum_t,
                       double* sim_q, double* sim_k, int8_t* Qq, float* q_scale, uint16_t* v_tiles, AttnStart start,
                       hipStream_t st);
// Token mean of K per (b,h) from the block sums.
hipError_t launch_k_mean(const double* ksum_t, const Shape& s, float* k_mean, hipStream_t st);
// INT8 quantization of K - k_mean.
hipError_t launch_quant_k(const void* K, const Shape& s, const float* k_mean, int8_t* Kq, float* k_scale,
                          hipStream_t st);
// Compressed logits S_hat = sm_scale * q k^T, fp64 [B,H,Tm,Tn]; causal: only tiles that some row sees are written.
hipError_t launch_logits(const double* pooled_q, const double* ksum_t, const Shape& s, float sm_scale, int causal,
                         double* logits, hipStream_t st);
// Softmax + TopCdf + overrides per mask row.
hipError_t launch_topcdf(const double* logits, const double* sim_q, const double* sim_k, const Shape& s,
                         const HeadParams& tau, const HeadParams& theta, int causal, uint8_t* mask,
                         hipStream_t st);
// Short calls: logits, TopCdf and the K quantization (mean included; none if Kq is null) in one launch.
hipError_t launch_predict_quant(const double* pooled_q, const double* ksum_t, const double* sim_q, const double* sim_k,
                                const void* K, const Shape& s, const HeadParams& tau, const HeadParams& theta,
                                float sm_scale, int causal, uint8_t* mask, int8_t* Kq, float* k_scale, hipStream_t st);
// V [B,H,N,d] (strided) -> per key block, d rows of 64 key slots in the order the P~V MFMA consumes.
hipError_t launch_v_tiles(const void* V, const Shape& s, uint16_t* v_tiles, hipStream_t st);
// lut[b,h,i,:] = the j with mask[b,h,i,j] != 0, ascending, then -1; lut_count[b,h,i] = how many.
hipError_t launch_mask_lut(const uint8_t* mask, const Shape& s, int32_t* lut, int32_t* lut_count, hipStream_t st);
// What an attention launch of this shape needs set, with its counters in ATTN_QUEUE_BYTES of device memory at `memory`
// that no other launch may use at the same time; launch_set_start sets it where no other kernel does.
hipError_t plan_start(const Shape& s, int causal, unsigned int* memory, unsigned long long* stats, AttnStart* start);
hipError_t launch_set_start(const AttnStart& start, hipStream_t st);
// The sparse flash loop (accumulates into stats).
hipError_t launch_attn(const void* Qp, const void* Kp, const float* q_scale, const float* k_scale,
                       const void* v_tiles, const float* v_scale, const Shape& s, const uint8_t* mask,
                       const HeadParams& lambda, float sm_scale, int causal, void* O, unsigned long long* stats,
                       const AttnStart& start, hipStream_t st);
// Calls of few Q blocks: the same loop with a 32-row group per workgroup (attn_split.hip), the same bits.
// attn_split_pays: a compute unit holds one workgroup of it, which runs a group's tiles in a half to two thirds of the
// time attn.hip needs; so it is worth it while every group has a unit (us, attn.hip / this, the attention alone, d = 64 and 128):
//   16 x 70 7.4 / 5.2, 8.5 / 6.0; 8 x 1024 16.8 / 9.7, 20.1 / 11.7; 2 x 4096 36.8 / 20.6, 43.6 / 28.1; 1 x 8192 49.8 / 27.5,
//   58.1 / 36.3; FP8 P~V 1 x 8192 52.5 / 26.3, 57.9 / 31.3; 16-bit Q K^T 57.0 / 31.7, 72.4 / 50.5.
// Beyond it, 12 x 1024 16.8 / 17.2, 20.4 / 21.0; 2 x 8192 50.2 / 50.2, 60.7 / 66.8; FP8 17.7 / 17.2, 20.7 / 18.9; 52.5 / 48.2, 59.4 /
// 58.2 but 51 x 320 10.2 / 12.3, 12.6 / 13.3; 16-bit Q K^T 20.5 / 21.0, 26.2 / 29.3; 57.7 / 55.5, 75.3 / 88.8.
// Causal groups start with the longest, and the second ones a unit gets can be the short ones.  Up to an eighth more groups
// than units that pays from rows of 4 blocks on (12 x 700 13.6 / 10.6, 15.9 / 12.3; 24 x 321 10.5 / 9.1, 11.8 / 10.5; rows of 2
// blocks 66 x 128 7.9 / 9.0, 9.1 / 10.7), up to half as many again from 8 blocks on (24 x 512 12.2 / 11.1, 14.2 / 12.7; 15 x 800
// 15.3 / 14.2, 17.9 / 17.6; shorter ones 34 x 321 10.5 / 11.0, 11.9 / 12.6) and up to two a unit where rows are long or an
// XCD's range is whole heads (5 x 3000 29.3 / 25.9, 34.3 / 32.1; 16 x 1024 17.6 / 14.1, 20.5 / 17.0; else 14 x 1100 18.1 / 18.7, 21.3 /
// 23.9; 10 x 1500 25.6 / 27.4 at 128; 128 x 128 8.1 / 9.7, 9.5 / 11.4); rows beyond 64 blocks 2 x 5000 x 128 45.2 / 46.8.  Not
// with the 16-bit Q K^T at d = 128, whose K tiles fill the LDS: 4 x 4096 64.6 / 65.8 with every block kept.
constexpr int SPLIT_MAX_TN = 128;    // key blocks its lists hold: a head of 256 row groups has no more
bool attn_split_pays(const Shape& s, int causal);
hipError_t launch_attn_split(const void* Qp, const void* Kp, const float* q_scale, const float* k_scale,
                             const void* v_tiles, const float* v_scale, const Shape& s, const uint8_t* mask,
                             const HeadParams& lambda, float scale, int causal, void* O, unsigned long long* stats,
                             hipStream_t st);
// FP8 form of V: per-(b,h,channel) |V| maxima (as fp32 bit patterns, zeroed here), scales amax/448, and
// E4M3 tiles in the operand order of the 32x32x64 MFMA.
hipError_t launch_v_tiles_fp8(const void* V, const Shape& s, unsigned char* tiles, float* v_scale,
                              uint32_t* amax_bits, hipStream_t st);

// out[b,h] = {sum|Oref - O|, sum|Oref|} in fp64 (overwritten; fixed summation order), both tensors laid out as the shape says.
hipError_t launch_rel_l1(const void* O, const void* Oref, const Shape& s, double* out, hipStream_t st);

// Order in which a Hilbert curve visits the row-major cells of a T x H x W grid (host; perm has T*H*W entries).
void hilbert_order_host(int T, int H, int W, int32_t* perm);
// Token gather by that order, or its inverse, on [off, off + L); other tokens are copied in place.
hipError_t launch_permute_tokens(const void* src, const Shape& s, const int32_t* perm, int L, int off, int inverse,
                                 void* dst, hipStream_t st);

}  // namespace sparge
