// Cross-lane reductions, 16-bit row unpacking and INT8 packing, and the INT8 quantization of one K block: shared by
// the passes over Q and K and by the launch that runs the block predictor beside the K quantization.
#pragma once
#include "common.hpp"

namespace sparge {

namespace {

// Cross-lane reductions on the vector ALU (DPP row operations and the lane-swap instructions, row_xchg and
// the swaps below) instead of ds_bpermute: the block statistics spend their time in the LDS pipeline otherwise.
// {own, partner's} in some order for the lanes ^16 or ^32: v_permlane16_swap / v_permlane32_swap of a register
// with its copy leave one of the two values in each result, which is all a commutative reduction needs
template <int PARTNER>
__device__ __forceinline__ void swap_pair(uint32_t v, uint32_t& a, uint32_t& b) {
    static_assert(PARTNER == 16 || PARTNER == 32, "no such exchange");
    if constexpr (PARTNER == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = r[0], b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = r[0], b = r[1];
    }
}
// v + (v of the partner lane)
template <int PARTNER>
__device__ __forceinline__ double add_partner(double v) {
    const uint32_t lo = static_cast<uint32_t>(__double2loint(v)), hi = static_cast<uint32_t>(__double2hiint(v));
    if constexpr (PARTNER == 16 || PARTNER == 32) {
        uint32_t l0, l1, h0, h1;
        swap_pair<PARTNER>(lo, l0, l1);
        swap_pair<PARTNER>(hi, h0, h1);
        return __hiloint2double(static_cast<int>(h0), static_cast<int>(l0)) +
               __hiloint2double(static_cast<int>(h1), static_cast<int>(l1));
    } else {
        return v + __hiloint2double(static_cast<int>(row_xchg<PARTNER>(hi)), static_cast<int>(row_xchg<PARTNER>(lo)));
    }
}
template <int PARTNER>
__device__ __forceinline__ float max_partner(float v) {
    if constexpr (PARTNER == 16 || PARTNER == 32) {
        uint32_t a, b;
        swap_pair<PARTNER>(__float_as_uint(v), a, b);
        return fmaxf(__uint_as_float(a), __uint_as_float(b));
    } else {
        return fmaxf(v, __uint_as_float(row_xchg<PARTNER>(__float_as_uint(v))));
    }
}
// Two values reduced at the price of one: the lanes whose number has bit PARTNER clear end up with
// a + (a of lane ^ PARTNER), the others with b + (b of lane ^ PARTNER).
template <int PARTNER>
__device__ __forceinline__ double scatter_sum(double a, double b) {
    if constexpr (PARTNER == 16 || PARTNER == 32) {
        // the swap moves a's upper half (odd rows) against b's lower half (even rows): no copies, no selects
        uint32_t l0, l1, h0, h1;
        if constexpr (PARTNER == 16) {
            const auto rl = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(__double2loint(a)),
                                                             static_cast<uint32_t>(__double2loint(b)), false, false);
            const auto rh = __builtin_amdgcn_permlane16_swap(static_cast<uint32_t>(__double2hiint(a)),
                                                             static_cast<uint32_t>(__double2hiint(b)), false, false);
            l0 = rl[0], l1 = rl[1], h0 = rh[0], h1 = rh[1];
        } else {
            const auto rl = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(__double2loint(a)),
                                                             static_cast<uint32_t>(__double2loint(b)), false, false);
            const auto rh = __builtin_amdgcn_permlane32_swap(static_cast<uint32_t>(__double2hiint(a)),
                                                             static_cast<uint32_t>(__double2hiint(b)), false, false);
            l0 = rl[0], l1 = rl[1], h0 = rh[0], h1 = rh[1];
        }
        return __hiloint2double(static_cast<int>(h0), static_cast<int>(l0)) +
               __hiloint2double(static_cast<int>(h1), static_cast<int>(l1));
    } else {
        static_assert(PARTNER == 1 || PARTNER == 2, "a true lane ^ PARTNER exchange is needed here");
        const bool up = (threadIdx.x & PARTNER) != 0;
        const double keep = up ? b : a, send = up ? a : b;
        return keep + __hiloint2double(static_cast<int>(row_xchg<PARTNER>(static_cast<uint32_t>(__double2hiint(send)))),
                                       static_cast<int>(row_xchg<PARTNER>(static_cast<uint32_t>(__double2loint(send)))));
    }
}
// v summed (maximized) over the aligned group of G lanes, G = 8, 16 or 64; every lane gets the result
template <int G>
__device__ __forceinline__ double group_sum(double v) {
    v = add_partner<1>(v);
    v = add_partner<2>(v);
    v = add_partner<7>(v);  // the quads agree by now: the mirrors do
    if constexpr (G >= 16) v = add_partner<15>(v);
    if constexpr (G == 64) {
        v = add_partner<16>(v);
        v = add_partner<32>(v);
    }
    return v;
}
template <int G>
__device__ __forceinline__ float group_max(float v) {
    v = max_partner<1>(v);
    v = max_partner<2>(v);
    v = max_partner<7>(v);
    if constexpr (G >= 16) v = max_partner<15>(v);
    return v;
}
template <int DT>
__device__ __forceinline__ void unpack8(const uint4& raw, float (&f)[8]) {
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = cvt16<DT>(static_cast<uint16_t>(w[e] & 0xFFFFu));
        f[2 * e + 1] = cvt16<DT>(static_cast<uint16_t>(w[e] >> 16));
    }
}

// x_hat = rint_half_even(x * r) packed as 8 int8 (fp32 multiply, single rounding, no contraction).
// Adding 1.5 * 2^23 to the rounded product rounds it to an integer, to nearest even, and leaves that
// integer in two's complement in the low mantissa bits (|x * r| <= 127): the low byte is x_hat.
__device__ __forceinline__ uint2 quant8(const float (&f)[8], float r) {
    uint32_t y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = __float_as_uint(f[e] * r + 12582912.0f);
    uint32_t out[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t lo = __builtin_amdgcn_perm(y[4 * h + 1], y[4 * h + 0], 0x0c0c0400u);  // bytes {y0, y1, 0, 0}
        const uint32_t hi = __builtin_amdgcn_perm(y[4 * h + 3], y[4 * h + 2], 0x0c0c0400u);
        out[h] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    }
    return make_uint2(out[0], out[1]);
}

// One 64-row K block by 256 threads (tid): K' = fp32(K) - mean, per-block amax, INT8.  mean: the 8 channels of the
// thread's chunk.  lds_amax: 4 floats of these 256 threads.  Every thread of the workgroup has to call this (it
// meets at a barrier); t >= Tn does nothing else.
template <int D, int DT>
__device__ __forceinline__ void quant_k_block(const uint16_t* __restrict__ base, const Shape& s, long long bh, int t,
                                              int tid, const float (&mean)[8], float* lds_amax,
                                              int8_t* __restrict__ Kq, float* __restrict__ k_scale) {
    constexpr int LPR = D / 8, RPW = 64 / LPR, RPS = 4 * RPW, NL = BK / RPS;
    const int lane = tid & 63, wave = tid >> 6;
    const int cchunk = lane % LPR, rsub = lane / LPR;
    const int row0 = t * BK;
    float x[NL][8];
    float amax = 0.f;
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        const int r = row0 + n * RPS + wave * RPW + rsub;
        uint4 raw = make_uint4(0u, 0u, 0u, 0u);
        const bool ok = r < s.N;
        if (ok) raw = *reinterpret_cast<const uint4*>(base + (long long)r * s.sn + cchunk * 8);
        unpack8<DT>(raw, x[n]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[n][e] = ok ? x[n][e] - mean[e] : 0.f;
            amax = fmaxf(amax, fabsf(x[n][e]));
        }
    }
    amax = group_max<16>(amax);
    amax = max_partner<16>(amax);
    amax = max_partner<32>(amax);
    if (lane == 0) lds_amax[wave] = amax;
    __syncthreads();
    if (t >= s.Tn) return;
    const float bmax = fmaxf(fmaxf(lds_amax[0], lds_amax[1]), fmaxf(lds_amax[2], lds_amax[3]));
    const float r = bmax > 0.f ? 127.0f / bmax : 0.f;
    if (tid == 0) k_scale[bh * s.Tn + t] = bmax > 0.f ? bmax / 127.0f : 0.f;
    int8_t* qbase = Kq + bh * (long long)s.N * D;
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        const int rr = row0 + n * RPS + wave * RPW + rsub;
        if (rr < s.N) *reinterpret_cast<uint2*>(qbase + (long long)rr * D + cchunk * 8) = quant8(x[n], r);
    }
}

}  // namespace

}  // namespace sparge
