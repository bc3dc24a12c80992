// Bandwidth-bound passes over Q and K (Alg. 1 lines 3-5):
//   block_stats  : one read of a 128-row Q block or 64-row K block -> pooled channel sums/means,
//                  block self-similarity CosSim, and (Q only) the per-block INT8 quantization.
//   k_mean       : per-(batch,head) token mean of K from the block sums.
//   quant_k      : second read of K -> INT8 of (K - mean) with per-block scales.
//   v_tiles      : V re-tiled per 64-key block into the operand order of the P~V matrix product.
// Thread mapping: a token row of d 16-bit values is covered by d/8 adjacent lanes holding 16 bytes
// each, so every global load instruction moves whole 128/256-byte rows; a lane keeps the same 8
// channels for all its rows, which makes channel sums per-lane accumulations.
#include "lanes.hpp"

namespace sparge {

namespace {

__device__ __forceinline__ double shfl_xor_f64(double v, int mask) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_xor(lo, mask);
    hi = __shfl_xor(hi, mask);
    return __hiloint2double(hi, lo);
}

// LDS of the block statistics; the other passes of the same launch use the same bytes.
template <int D>
struct StatsLds {
    double raw[4][D], hat[4][D];
    double sq[4];
    double inv[4][64];
    float amax[4];
};

// One workgroup (256 threads) per block of ROWS tokens: block t of (batch, head) bh, whose rows start at base.
//   KSIDE: sums go out transposed and unscaled ([B,H,d,Tn], needed exactly for the K mean), otherwise means go out
//   as [B,H,Tm,d].
//   QUANT: the block is quantized in place from registers (Q side only).
//   STATS: without it nothing of the above but what the quantization needs: the K side's sums (for the mean), in the
//   same order; the fp64 arithmetic of the norms and of the self-similarity is what bounds the full version.
template <int D, int DT, int ROWS, bool KSIDE, bool QUANT, bool STATS>
__device__ __forceinline__ void block_stats(StatsLds<D>& lds, const uint16_t* __restrict__ base, const Shape& s,
                                            const long long bh, const int t, double* __restrict__ pooled,
                                            double* __restrict__ sim, int8_t* __restrict__ Xq,
                                            float* __restrict__ scale) {
    constexpr int LPR = D / 8;        // lanes per token row
    constexpr int RPW = 64 / LPR;     // rows per wave-wide load
    constexpr int RPS = 4 * RPW;      // rows per sweep of the 4 waves
    constexpr int NL = ROWS / RPS;    // loads per lane
    const int T = KSIDE ? s.Tn : s.Tm;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cchunk = lane % LPR, rsub = lane / LPR;
    const int row0 = t * ROWS;
    static_assert(NL * RPW <= 64, "a wave's rows must fit one lane each");
    auto& lds_raw = lds.raw;
    auto& lds_hat = lds.hat;
    auto& lds_amax = lds.amax;
    auto& lds_sq = lds.sq;
    auto& lds_inv = lds.inv;

    uint4 raw[NL];
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        const int r = row0 + n * RPS + wave * RPW + rsub;
        raw[n] = make_uint4(0u, 0u, 0u, 0u);
        if (r < s.N) raw[n] = *reinterpret_cast<const uint4*>(base + (long long)r * s.sn + cchunk * 8);
    }

    double sraw[8], shat[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sraw[e] = shat[e] = 0.0;
    float amax = 0.f;
    // squared norm of every row of this wave (NL * RPW of them), one value per row in LDS
    double nsq[NL];
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        float f[8];
        unpack8<DT>(raw[n], f);
        nsq[n] = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double x = static_cast<double>(f[e]);
            if constexpr (STATS) nsq[n] = __builtin_fma(x, x, nsq[n]);  // x * x is exact in fp64 (16-bit inputs): same result as mul + add
            if constexpr (QUANT) amax = fmaxf(amax, fabsf(f[e]));
        }
    }
    // The LPR lanes of a row are summed with the first steps halving the number of values: after them
    // the lane with bits (p, q) = (lane & 1, lane >> 1 & 1) works on the rows n = i + NQ q + NH p only.
    if constexpr (STATS) {
        static_assert(NL == 2 || NL == 4 || NL == 8, "row count per lane");
        constexpr int NH = NL / 2, NQ = NL >= 4 ? NL / 4 : 1;
        double w1[NH];
#pragma unroll
        for (int i = 0; i < NH; ++i) w1[i] = scatter_sum<1>(nsq[i], nsq[i + NH]);
        const int p = lane & 1, q = (lane >> 1) & 1;
        if constexpr (NL >= 4) {
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                double w = scatter_sum<2>(w1[i], w1[i + NQ]);
                w = add_partner<4>(w);  // lanes of a quad hold different rows from here on: true ^4, ^8 only
                if constexpr (LPR == 16) w = add_partner<8>(w);
                if (cchunk < 4) lds_inv[wave][(i + NQ * q + NH * p) * RPW + rsub] = w;
            }
        } else {
            double w = add_partner<2>(w1[0]);
            w = add_partner<4>(w);
            if constexpr (LPR == 16) w = add_partner<8>(w);
            if (cchunk < 2) lds_inv[wave][p * RPW + rsub] = w;
        }
    }
    // 1 / |row|: the fp64 square root and division are the expensive part, so each row's is evaluated by
    // one lane only (a wave owns at most 64 rows) and handed to the lanes of that row through LDS
    // (the exchange stays inside a wave, whose LDS accesses complete in program order: the wave barriers
    // only keep the compiler from moving accesses across the hand-over points)
    __builtin_amdgcn_wave_barrier();
    if (STATS && lane < NL * RPW) {
        const double nsq = lds_inv[wave][lane];
        lds_inv[wave][lane] = nsq > 0.0 ? 1.0 / sqrt(nsq) : 0.0;
    }
    __builtin_amdgcn_wave_barrier();
    if constexpr (STATS || KSIDE) {
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            float f[8];
            unpack8<DT>(raw[n], f);
            const double inv = STATS ? lds_inv[wave][n * RPW + rsub] : 0.0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const double x = static_cast<double>(f[e]);
                sraw[e] += x;
                if constexpr (STATS) shat[e] = __builtin_fma(x, inv, shat[e]);
            }
        }
    }
    // Combine the lanes that hold the same channels (different rows of the wave-wide load).  Lane bits 5
    // and 4 each halve the 16 sums a lane works on: lane bit 5 selects raw sums / normalized sums, lane
    // bit 4 the channels 0..3 / 4..7 of the lane's chunk.  (d = 64: lane bit 3 is reduced last, in full.)
    if constexpr (STATS || KSIDE) {
        double h8[8], h4[4];
#pragma unroll
        for (int e = 0; e < 8; ++e) h8[e] = scatter_sum<32>(sraw[e], shat[e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) h4[e] = scatter_sum<16>(h8[e], h8[e + 4]);
        if constexpr (LPR == 8) {
#pragma unroll
            for (int e = 0; e < 4; ++e) h4[e] = add_partner<8>(h4[e]);
        }
        if (LPR == 16 || (lane & 8) == 0) {
            double* dst = (lane & 32) ? lds_hat[wave] : lds_raw[wave];
            const int c0 = cchunk * 8 + ((lane & 16) ? 4 : 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[c0 + e] = h4[e];
        }
    }
    if constexpr (QUANT) {
        amax = max_partner<32>(amax);
        amax = max_partner<16>(amax);
        if constexpr (LPR == 8) amax = max_partner<8>(amax);
        amax = group_max<LPR>(amax);
    }
    if (lane == 0) lds_amax[wave] = amax;
    __syncthreads();

    if constexpr (STATS || KSIDE) {
        const int cnt = min(ROWS, s.N - row0);
        if (threadIdx.x < D) {
            const int c = threadIdx.x;
            const double rsum = ((lds_raw[0][c] + lds_raw[1][c]) + lds_raw[2][c]) + lds_raw[3][c];
            if (KSIDE) pooled[(bh * D + c) * T + t] = rsum;
            else pooled[(bh * T + t) * D + c] = rsum / static_cast<double>(cnt);
            if constexpr (STATS) {
                const double hsum = ((lds_hat[0][c] + lds_hat[1][c]) + lds_hat[2][c]) + lds_hat[3][c];
                double sq = hsum * hsum;
                sq = group_sum<64>(sq);
                if (lane == 0) lds_sq[wave] = sq;
            }
        }
        if constexpr (STATS) {
            __syncthreads();
            if (threadIdx.x == 0) {
                double tot = lds_sq[0];
                if (D > 64) tot += lds_sq[1];
                sim[bh * T + t] = tot / (static_cast<double>(cnt) * static_cast<double>(cnt));
            }
        }
    }

    if constexpr (QUANT) {
        const float bmax = fmaxf(fmaxf(lds_amax[0], lds_amax[1]), fmaxf(lds_amax[2], lds_amax[3]));
        const float r = bmax > 0.f ? 127.0f / bmax : 0.f;
        if (threadIdx.x == 0) scale[bh * T + t] = bmax > 0.f ? bmax / 127.0f : 0.f;
        int8_t* qbase = Xq + bh * (long long)s.N * D;
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            const int rr = row0 + n * RPS + wave * RPW + rsub;
            if (rr < s.N) {
                float f[8];
                unpack8<DT>(raw[n], f);
                *reinterpret_cast<uint2*>(qbase + (long long)rr * D + cchunk * 8) = quant8(f, r);
            }
        }
    }
}

// One workgroup per (b, h, 4 channels): wave w reduces channel 4*blockIdx.x + w; lanes stride over the
// key blocks and combine in a fixed butterfly, so the sum does not depend on scheduling.
template <int D>
__global__ __launch_bounds__(256) void k_mean_kernel(const double* __restrict__ ksum_t, Shape s,
                                                      float* __restrict__ k_mean) {
    const long long bh = (long long)blockIdx.z * s.H + blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = blockIdx.x * 4 + wave;
    const double* row = ksum_t + (bh * D + c) * s.Tn;
    double acc = 0.0;
    for (int j = lane; j < s.Tn; j += 64) acc += row[j];
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) acc += shfl_xor_f64(acc, m);
    if (lane == 0) k_mean[bh * D + c] = static_cast<float>(acc / static_cast<double>(s.N));
}

// One workgroup per 64-row K block, the mean from memory.
template <int D, int DT>
__global__ __launch_bounds__(256) void quant_k_kernel(const uint16_t* __restrict__ K, Shape s,
                                                       const float* __restrict__ k_mean,
                                                       int8_t* __restrict__ Kq, float* __restrict__ k_scale) {
    const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const long long bh = (long long)b * s.H + h;
    const int cchunk = threadIdx.x % (D / 8);
    __shared__ float lds_amax[4];
    float mean[8];
    {
        const float4 m0 = *reinterpret_cast<const float4*>(k_mean + bh * D + cchunk * 8);
        const float4 m1 = *reinterpret_cast<const float4*>(k_mean + bh * D + cchunk * 8 + 4);
        mean[0] = m0.x; mean[1] = m0.y; mean[2] = m0.z; mean[3] = m0.w;
        mean[4] = m1.x; mean[5] = m1.y; mean[6] = m1.z; mean[7] = m1.w;
    }
    quant_k_block<D, DT>(K + b * s.sb + h * s.sh, s, bh, t, static_cast<int>(threadIdx.x), mean, lds_amax, Kq, k_scale);
}

// One workgroup per 64-key block: tile[c][slot] = V[key(slot)][c], 64 slots per channel row.
// Within each group of 16 keys the slot order is {0..3, 8..11, 4..7, 12..15}: the order in which
// the 32x32 MFMA accumulator of S^T hands a lane its keys, so P~ feeds the P~V product from
// registers.  Keys >= N are written as zeros.
template <int D>
struct VTileLds {
    static constexpr int PITCH = D + 8;  // 16-bit elements; keeps the column reads spread over LDS banks
    uint16_t v[BK * PITCH];
};
template <int D>
__device__ __forceinline__ void v_tile(VTileLds<D>& tile, const uint16_t* __restrict__ base, const Shape& s,
                                       const long long bh, const int j, uint16_t* __restrict__ tiles) {
    constexpr int PITCH = VTileLds<D>::PITCH;
    uint16_t* const lds = tile.v;
    constexpr int CPR = D / 8;  // 16-byte chunks per key row
    constexpr int NL = BK * CPR / 256;
    uint4 v[NL];
#pragma unroll
    for (int n = 0; n < NL; ++n) {   // (loads without conditions, all in flight before the first goes to LDS)
        const int idx = threadIdx.x + n * 256, row = idx / CPR, col = idx % CPR;
        v[n] = *reinterpret_cast<const uint4*>(base + (long long)min(j * BK + row, s.N - 1) * s.sn + col * 8);
    }
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        const int idx = threadIdx.x + n * 256, row = idx / CPR, col = idx % CPR;
        *reinterpret_cast<uint4*>(&lds[row * PITCH + col * 8]) = j * BK + row < s.N ? v[n] : make_uint4(0u, 0u, 0u, 0u);
    }
    __syncthreads();
    uint16_t* out = tiles + (bh * s.Tn + j) * (long long)(D * BK);
    for (int idx = threadIdx.x; idx < D * 8; idx += 256) {
        const int c = idx / 8, sc = idx % 8;  // channel row, chunk of 8 slots
        uint32_t w[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            uint32_t pair = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int slot = sc * 8 + e2 * 2 + q;
                const int g = slot >> 4, sl = slot & 15;
                const int key = g * 16 + 8 * ((sl & 7) >> 2) + 4 * (sl >> 3) + (sl & 3);
                pair |= static_cast<uint32_t>(lds[key * PITCH + c]) << (16 * q);
            }
            w[e2] = pair;
        }
        *reinterpret_cast<uint4*>(out + c * BK + sc * 8) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

template <int D>
__global__ __launch_bounds__(256) void v_tiles_kernel(const uint16_t* __restrict__ V, Shape s,
                                                       uint16_t* __restrict__ tiles) {
    __shared__ __align__(16) VTileLds<D> tile;
    const int j = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    v_tile<D>(tile, V + b * s.sb + h * s.sh, s, (long long)b * s.H + h, j, tiles);
}

// Which K block the workgroup (bh, t) of the launch takes.  The channel sums are [bh][d][Tn] doubles, one from each block, so
// 16 blocks side by side fill a 128-byte line, and it should be one XCD (workgroup numbers equal modulo 8) whose L2 does.
// Each XCD takes an eighth of a head's blocks; heads of fewer than 16 blocks share lines among channels instead, and
// 128 consecutive blocks are dealt out 16 to an XCD across heads.  Measured against no reordering, us: predictor 456 / 478 at
// 32 x 65536 x 128, 105 / 110 at 24 x 22272 x 128, 73.0 / 76.7 at 512 x 1024 x 128 (16 blocks), sparge_quantize 120 / 125 at
// 2048 x 200 x 128 (4 blocks).  Dealing out across heads everywhere costs three divisions per workgroup, 470 and 106 us.
constexpr int K_BLOCKS_OF_ITS_OWN = 16;
__device__ __forceinline__ void k_block_of(const Shape& s, int& bh, int& t) {
    if (s.Tn >= K_BLOCKS_OF_ITS_OWN) {
        if (t < (s.Tn & ~7)) t = (t & 7) * (s.Tn >> 3) + (t >> 3);
    } else {
        const int id = bh * s.Tn + t;
        if (id < ((s.B * s.H * s.Tn) & ~127)) {
            const int to = (id & ~127) + (id & 7) * 16 + ((id & 127) >> 3);
            bh = to / s.Tn, t = to % s.Tn;
        }
    }
}

template <int D, int DT, int ROWS, bool KSIDE, bool QUANT, bool STATS>
__global__ __launch_bounds__(256) void block_stats_kernel(const uint16_t* __restrict__ X, Shape s,
                                                          double* __restrict__ pooled, double* __restrict__ sim,
                                                          int8_t* __restrict__ Xq, float* __restrict__ scale,
                                                          AttnStart start) {
    __shared__ StatsLds<D> lds;
    int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    if constexpr (KSIDE) {
        int bh = b * s.H + h;
        k_block_of(s, bh, t);
        if (s.Tn < K_BLOCKS_OF_ITS_OWN) b = bh / s.H, h = bh % s.H;
    } else if (t + h + b == 0) {
        set_start(start, 0, 1);
    }
    block_stats<D, DT, ROWS, KSIDE, QUANT, STATS>(lds, X + b * s.sb + h * s.sh, s, (long long)b * s.H + h, t, pooled, sim,
                                                  Xq, scale);
}

// The statistics of all Q blocks (with their INT8 form if QUANT) and all K blocks, and the V tiles where the caller
// wants them here (v_tiles not null), in one launch: none of them waits for another, and a launch of its own for
// each cost a small call more than the work.  Workgroup order: Q blocks (the longest), K blocks, V blocks.
template <int D, int DT, bool QUANT>
__global__ __launch_bounds__(256) void prep_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                   const uint16_t* __restrict__ V, Shape s,
                                                   double* __restrict__ pooled_q, double* __restrict__ ksum_t,
                                                   double* __restrict__ sim_q, double* __restrict__ sim_k,
                                                   int8_t* __restrict__ Qq, float* __restrict__ q_scale,
                                                   uint16_t* __restrict__ v_tiles, AttnStart start) {
    __shared__ __align__(16) union {
        StatsLds<D> stats;
        VTileLds<D> tile;
    } lds;
    const int nq = s.B * s.H * s.Tm, nk = s.B * s.H * s.Tn;
    int id = blockIdx.x;
    if (id == 0) set_start(start, 0, 1);
    auto at = [&](const uint16_t* X, int bh) { return X + (bh / s.H) * s.sb + (bh % s.H) * s.sh; };
    if (id < nq) {
        const int bh = id / s.Tm;
        block_stats<D, DT, BQ, false, QUANT, true>(lds.stats, at(Q, bh), s, bh, id % s.Tm, pooled_q, sim_q, Qq, q_scale);
        return;
    }
    id -= nq;
    if (id < nk) {
        int bh = id / s.Tn, t = id % s.Tn;
        k_block_of(s, bh, t);
        block_stats<D, DT, BK, true, false, true>(lds.stats, at(K, bh), s, bh, t, ksum_t, sim_k, nullptr, nullptr);
        return;
    }
    id -= nk;
    const int bh = id / s.Tn;
    v_tile<D>(lds.tile, at(V, bh), s, bh, id % s.Tn, v_tiles);
}

}  // namespace

#define SPARGE_DISPATCH_D_DT(s, CALL)                                              \
    if ((s).d == 64 && (s).dtype == SPARGE_F16) { CALL(64, SPARGE_F16) }           \
    else if ((s).d == 64 && (s).dtype == SPARGE_BF16) { CALL(64, SPARGE_BF16) }    \
    else if ((s).d == 128 && (s).dtype == SPARGE_F16) { CALL(128, SPARGE_F16) }    \
    else if ((s).d == 128 && (s).dtype == SPARGE_BF16) { CALL(128, SPARGE_BF16) }  \
    else return hipErrorInvalidValue;

hipError_t launch_block_stats(const void* Q, const void* K, const Shape& s, double* pooled_q, double* ksum_t,
                              double* sim_q, double* sim_k, int8_t* Qq, float* q_scale, AttnStart start, hipStream_t st) {
    const dim3 gq(s.Tm, s.H, s.B), gk(s.Tn, s.H, s.B);
    const uint16_t *q = static_cast<const uint16_t*>(Q), *k = static_cast<const uint16_t*>(K);
    const AttnStart none{};
#define CALL(D, DT)                                                                                                   \
    if (!sim_q) {                                                                                                     \
        hipLaunchKernelGGL((block_stats_kernel<D, DT, BQ, false, true, false>), gq, dim3(256), 0, st, q, s, pooled_q, \
                           sim_q, Qq, q_scale, start);                                                                \
        hipLaunchKernelGGL((block_stats_kernel<D, DT, BK, true, false, false>), gk, dim3(256), 0, st, k, s, ksum_t,   \
                           sim_k, (int8_t*)nullptr, (float*)nullptr, none);                                           \
    } else {                                                                                                          \
        if (Qq) hipLaunchKernelGGL((block_stats_kernel<D, DT, BQ, false, true, true>), gq, dim3(256), 0, st, q, s,    \
                                   pooled_q, sim_q, Qq, q_scale, start);                                              \
        else hipLaunchKernelGGL((block_stats_kernel<D, DT, BQ, false, false, true>), gq, dim3(256), 0, st, q, s,      \
                                pooled_q, sim_q, Qq, q_scale, start);                                                 \
        hipLaunchKernelGGL((block_stats_kernel<D, DT, BK, true, false, true>), gk, dim3(256), 0, st, k, s, ksum_t,    \
                           sim_k, (int8_t*)nullptr, (float*)nullptr, none);                                           \
    }
    SPARGE_DISPATCH_D_DT(s, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_prep(const void* Q, const void* K, const void* V, const Shape& s, double* pooled_q, double* ksum_t,
                       double* sim_q, double* sim_k, int8_t* Qq, float* q_scale, uint16_t* v_tiles, AttnStart start,
                       hipStream_t st) {
    if (!short_call(s)) return hipErrorInvalidValue;
    const dim3 grid(s.B * s.H * (s.Tm + (v_tiles ? 2 : 1) * s.Tn));
    const uint16_t *q = static_cast<const uint16_t*>(Q), *k = static_cast<const uint16_t*>(K),
                   *v = static_cast<const uint16_t*>(V);
#define CALL(D, DT)                                                                                                  \
    if (Qq) hipLaunchKernelGGL((prep_kernel<D, DT, true>), grid, dim3(256), 0, st, q, k, v, s, pooled_q, ksum_t,     \
                               sim_q, sim_k, Qq, q_scale, v_tiles, start);                                           \
    else hipLaunchKernelGGL((prep_kernel<D, DT, false>), grid, dim3(256), 0, st, q, k, v, s, pooled_q, ksum_t,       \
                            sim_q, sim_k, Qq, q_scale, v_tiles, start);
    SPARGE_DISPATCH_D_DT(s, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_k_mean(const double* ksum_t, const Shape& s, float* k_mean, hipStream_t st) {
    dim3 grid(s.d / 4, s.H, s.B);
    if (s.d == 64) hipLaunchKernelGGL((k_mean_kernel<64>), grid, dim3(256), 0, st, ksum_t, s, k_mean);
    else hipLaunchKernelGGL((k_mean_kernel<128>), grid, dim3(256), 0, st, ksum_t, s, k_mean);
    return hipGetLastError();
}

hipError_t launch_quant_k(const void* K, const Shape& s, const float* k_mean, int8_t* Kq, float* k_scale,
                          hipStream_t st) {
    dim3 grid(s.Tn, s.H, s.B);
    const uint16_t* X = static_cast<const uint16_t*>(K);
#define CALL(D, DT) \
    hipLaunchKernelGGL((quant_k_kernel<D, DT>), grid, dim3(256), 0, st, X, s, k_mean, Kq, k_scale);
    SPARGE_DISPATCH_D_DT(s, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_v_tiles(const void* V, const Shape& s, uint16_t* v_tiles, hipStream_t st) {
    dim3 grid(s.Tn, s.H, s.B);
    const uint16_t* X = static_cast<const uint16_t*>(V);
    if (s.d == 64) hipLaunchKernelGGL((v_tiles_kernel<64>), grid, dim3(256), 0, st, X, s, v_tiles);
    else hipLaunchKernelGGL((v_tiles_kernel<128>), grid, dim3(256), 0, st, X, s, v_tiles);
    return hipGetLastError();
}

}  // namespace sparge
