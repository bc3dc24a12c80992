// Stage-1 predictor after the block statistics (Alg. 1 lines 5-6; Sec. 3.2):
//   logits : S_hat = sm_scale * q k^T on the pooled tokens, fp64 (tiny next to the attention itself)
//   topcdf : per mask row: -inf columns, softmax, TopCdf(tau) by bracketing the cut in the ranking (rows beyond
//            2048 key blocks: by an in-LDS bitonic sort and a prefix sum), fix-block overrides, causal rules.
//   short calls: both in one launch, beside the K quantization (predict_quant_kernel).
// All arithmetic is fp64 so that block decisions agree with an fp64 reference except for
// statistics that sit within ~1e-13 of a threshold.
#include "lanes.hpp"

namespace sparge {

namespace {

__device__ __forceinline__ double shfl_xor_f64(double v, int mask) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_xor(lo, mask);
    hi = __shfl_xor(hi, mask);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double shfl_up_f64(double v, int delta) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_up(lo, delta);
    hi = __shfl_up(hi, delta);
    return __hiloint2double(hi, lo);
}

// A wave-uniform fp64 value, moved to scalar registers.
__device__ __forceinline__ double uniform_f64(double v) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)), __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// Key blocks that mask row i has to rank: all of them, or (causal) those up to the end of its own Q block.
__device__ __forceinline__ int visible_blocks(const Shape& s, int i, int causal) {
    static_assert(BQ == 2 * BK, "a Q block ends with the second key block of its own");
    return causal ? min(s.Tn, 2 * i + 2) : s.Tn;
}

// Compressed logits as an fp64 matrix product on the matrix cores: a wave computes RT x 16 pooled query rows x 64
// key blocks with v_mfma_f64_16x16x4_f64 (operands: lane = row or column + 16 * k; result register r of a
// lane = row 4 r + lane / 16, column lane % 16).  The pooled queries are row-major, the key sums
// transposed ([d][Tn]), so the B operand loads are lane-coalesced; both operands stay L2-resident and go
// straight from the caches into the operands, RT + 4 loads for 4 RT matrix instructions per step of 4 channels
// (RT is chosen at launch).  What bounds it is the matrix instruction itself: one per 100-115 cycles and SIMD however many
// waves offer it (counters: waves wait for issue 86 % of the time, for memory 7 %), half the nominal rate.
typedef double v4d __attribute__((ext_vector_type(4)));
template <int D, int RT>
__global__ __launch_bounds__(256) void logits_kernel(const double* __restrict__ pooled_q,
                                                      const double* __restrict__ ksum_t, Shape s,
                                                      double sm_scale, int causal, double* __restrict__ logits) {
    const long long bh = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = (blockIdx.y * 4 + wave) * 16 * RT, j0 = blockIdx.x * 64;
    if (i0 >= s.Tm || j0 >= visible_blocks(s, i0 + 16 * RT - 1, causal)) return;   // (nobody reads what no row sees)
    const int l16 = lane & 15, kk = lane >> 4;
    const double* qrow[RT];
#pragma unroll
    for (int u = 0; u < RT; ++u)   // rows past Tm: a valid row, not stored
        qrow[u] = pooled_q + (bh * s.Tm + min(i0 + 16 * u + l16, s.Tm - 1)) * D + kk;
    const double* kcol[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) kcol[t] = ksum_t + bh * D * s.Tn + (long long)kk * s.Tn + min(j0 + 16 * t + l16, s.Tn - 1);
    v4d acc[RT][4];
#pragma unroll
    for (int u = 0; u < RT; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[u][t] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < D; c += 4) {
        double a[RT], bcol[4];
#pragma unroll
        for (int u = 0; u < RT; ++u) a[u] = qrow[u][c];
#pragma unroll
        for (int t = 0; t < 4; ++t) bcol[t] = kcol[t][(long long)c * s.Tn];
#pragma unroll
        for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], bcol[t], acc[u][t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int j = j0 + 16 * t + l16;
        if (j >= s.Tn) continue;
        const double cnt = static_cast<double>(min(BK, s.N - j * BK));
#pragma unroll
        for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + 16 * u + 4 * r + kk;
                if (i < s.Tm) logits[(bh * s.Tm + i) * s.Tn + j] = sm_scale * (acc[u][t][r] / cnt);
            }
    }
}

__device__ __forceinline__ double block_reduce(double v, bool is_max, double* scratch) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const double o = shfl_xor_f64(v, m);
        v = is_max ? fmax(v, o) : v + o;
    }
    __syncthreads();
    if (lane == 0) scratch[wave] = v;
    __syncthreads();
    double r = scratch[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) r = is_max ? fmax(r, scratch[w]) : r + scratch[w];
    return r;
}

// One workgroup per mask row (b, h, i).  npad = power of two >= max(Tn, 2).
__global__ __launch_bounds__(256) void topcdf_kernel(const double* __restrict__ logits,
                                                      const double* __restrict__ sim_q,
                                                      const double* __restrict__ sim_k, Shape s,
                                                      HeadParams tau_h, HeadParams theta_h, int causal,
                                                      int npad, uint8_t* __restrict__ mask) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* keys = reinterpret_cast<double*>(smem);                      // [npad] probabilities by key block
    unsigned long long* skey = reinterpret_cast<unsigned long long*>(keys + npad);  // [npad] sort keys
    uint8_t* flag = reinterpret_cast<uint8_t*>(skey + npad);             // [npad]
    __shared__ double scratch[4];
    __shared__ double wave_tot[4];

    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const long long bh = (long long)b * s.H + h;
    const int tid = threadIdx.x;
    const int op = s.operand(static_cast<int>(bh)), par = s.param(static_cast<int>(bh), h);   // (Shape: settings of one launch)
    const double tau = static_cast<double>(tau_h.v[par]);
    const double theta = static_cast<double>(theta_h.v[par]);
    const double* row = logits + ((long long)op * s.Tm + i) * s.Tn;
    const double* sk = sim_k + (long long)op * s.Tn;
    const double NEG = -__builtin_inf();

    // A query block that is not self-similar keeps every (visible) key block: nothing to rank.
    if (sim_q[(long long)op * s.Tm + i] < theta) {
        uint8_t* out_row = mask + (bh * s.Tm + i) * s.Tn;
        for (int j = tid; j < s.Tn; j += 256) out_row[j] = (causal && j * BK > i * BQ + (BQ - 1)) ? 0 : 1;
        return;
    }

    // 1. masked logits and their maximum
    double mx = NEG;
    for (int j = tid; j < npad; j += 256) {
        double x = NEG;
        if (j < visible_blocks(s, i, causal)) {
            x = row[j];
            if (sk[j] < theta) x = NEG;
        }
        keys[j] = x;
        mx = fmax(mx, x);
    }
    mx = block_reduce(mx, true, scratch);
    // 2. softmax numerators and their sum
    double z = 0.0;
    for (int j = tid; j < npad; j += 256) {
        const double x = keys[j];
        const double e = (x == NEG) ? 0.0 : exp(x - mx);
        keys[j] = e;
        z += e;
    }
    z = block_reduce(z, false, scratch);
    double tot = 0.0;
    for (int j = tid; j < npad; j += 256) {
        double p = -1.0;  // padding ranks after every probability
        if (j < s.Tn) {
            p = z > 0.0 ? keys[j] / z : 0.0;
            tot += p;
        }
        keys[j] = p;
        // Sort key: the probability's bit pattern (non-negative doubles order like integers) with its low
        // 16 mantissa bits replaced by 0xFFFF - j: one 64-bit comparison ranks by (value descending, index
        // ascending).  Values closer than 2^-36 relative may swap ranks; that moves a prefix mass by less
        // than 2^-36, far inside the band in which a decision counts as a tie.
        skey[j] = p < 0.0 ? 0ull
                          : ((static_cast<unsigned long long>(__double_as_longlong(p)) & ~0xFFFFull) |
                             static_cast<unsigned long long>(0xFFFF - j));
        flag[j] = 0;
    }
    tot = block_reduce(tot, false, scratch);  // also orders the LDS writes before the sort

    // 3. bitonic sort: rank order = (value descending, index ascending).  Each wave owns a quarter of the
    // array: every compare-exchange at a distance inside a quarter touches the wave's own elements only,
    // and a wave's LDS accesses complete in program order, so those stages need no workgroup barrier
    // (the wave barrier only pins the compiler's order).  Only the few stages that reach across quarters
    // are bracketed by barriers.
    auto exchange = [&](int lo, int jj, int k) {
        const int hi = lo + jj;
        const unsigned long long ka = skey[lo], kb = skey[hi];
        const bool a_first = ka > kb;   // keys are distinct except among the padding
        const bool want_a_first = (lo & k) == 0;
        if (a_first != want_a_first && ka != kb) {
            skey[lo] = kb;
            skey[hi] = ka;
        }
    };
    const int epw = npad >> 2;  // elements per wave
    if (epw >= 128) {
        const int lane_ = tid & 63, seg = (tid >> 6) * epw;
        for (int k = 2; k <= npad; k <<= 1) {
            int jj = k >> 1;
            if (jj >= epw) {
                __syncthreads();
                for (; jj >= epw; jj >>= 1) {
                    for (int t = tid; t < (npad >> 1); t += 256) exchange(2 * jj * (t / jj) + (t % jj), jj, k);
                    __syncthreads();
                }
            }
            for (; jj > 0; jj >>= 1) {
                for (int t = lane_; t < (epw >> 1); t += 64) exchange(seg + 2 * jj * (t / jj) + (t % jj), jj, k);
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
    } else {
        for (int k = 2; k <= npad; k <<= 1) {
            for (int jj = k >> 1; jj > 0; jj >>= 1) {
                for (int t = tid; t < (npad >> 1); t += 256) exchange(2 * jj * (t / jj) + (t % jj), jj, k);
                __syncthreads();
            }
        }
    }

    // 4. exclusive prefix mass per rank; rank r is kept iff mass before it < tau * total
    const int per = (npad + 255) / 256;  // consecutive ranks per thread
    const int r0 = tid * per;
    double local = 0.0;
    auto rank_index = [&](int r) { return 0xFFFF - static_cast<int>(skey[r] & 0xFFFFull); };
    auto rank_value = [&](int r) { return skey[r] ? keys[rank_index(r)] : 0.0; };   // padding ranks last, mass 0
    for (int r = r0; r < min(r0 + per, npad); ++r) local += rank_value(r);
    // inclusive scan of `local` over the 256 threads
    const int lane = tid & 63, wave = tid >> 6;
    double incl = local;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double o = shfl_up_f64(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    double before = incl - local;
    for (int w = 0; w < wave; ++w) before += wave_tot[w];
    const double thresh = tau * tot;
    for (int r = r0; r < min(r0 + per, npad); ++r) {
        const double p = rank_value(r);
        if (p > 0.0 && before < thresh) flag[rank_index(r)] = 1;
        before += p;
    }
    __syncthreads();

    // 5. fix-block overrides and causal rules, then the row goes out
    const bool fix_q = sim_q[(long long)op * s.Tm + i] < theta;
    uint8_t* out = mask + (bh * s.Tm + i) * s.Tn;
    for (int j = tid; j < s.Tn; j += 256) {
        uint8_t m = flag[j];
        if (fix_q || sk[j] < theta) m = 1;
        if (causal) {
            if (j * BK > i * BQ + (BQ - 1)) m = 0;
            if (j == (i * BQ) / BK) m = 1;
        }
        out[j] = m;
    }
}

// maximum over the wave (every lane gets it)
template <int PARTNER>
__device__ __forceinline__ double max_of_partner(double v) {
    const uint32_t lo = static_cast<uint32_t>(__double2loint(v)), hi = static_cast<uint32_t>(__double2hiint(v));
    if constexpr (PARTNER >= 16) {
        uint32_t l0, l1, h0, h1;
        swap_pair<PARTNER>(lo, l0, l1);
        swap_pair<PARTNER>(hi, h0, h1);
        return fmax(__hiloint2double(static_cast<int>(h0), static_cast<int>(l0)),
                    __hiloint2double(static_cast<int>(h1), static_cast<int>(l1)));
    } else {
        return fmax(v, __hiloint2double(static_cast<int>(row_xchg<PARTNER>(hi)), static_cast<int>(row_xchg<PARTNER>(lo))));
    }
}
__device__ __forceinline__ double wave_max(double v) {
    v = max_of_partner<1>(v);
    v = max_of_partner<2>(v);
    v = max_of_partner<7>(v);
    v = max_of_partner<15>(v);
    v = max_of_partner<16>(v);
    return max_of_partner<32>(v);
}

// TopCdf of one mask row by one wave, without sorting the row: an entry is kept if the mass ranked before it is below
// the threshold, so one cut in the ranking decides the row.  Keys (see topcdf_kernel) rank the entries by one 64-bit
// comparison; lane L holds those of key blocks 64 e + L.  The cut is bracketed between two keys -- the mass from `lo` on
// reaches the threshold, the mass from `hi` on does not -- and the bracket halved until at most FEW entries lie in it; those
// are ranked one by one, two lanes an entry.  The first probe is the smallest probability the cut can have when nothing else is
// known (all that ranks from the cut on is more than (1 - tau) of the mass), which leaves the few octaves below the row's
// maximum.  Once two probes have left no entry out, the bracket shrinks to the keys in it; entries that are equal up to
// their index then (repeated or padded tokens: halving alone would take 50 probes to tell them apart) rank by it at once.
// What bounds it is the vector ALU (16 rows a SIMD at 32 x 65536): a probe costs EPL comparisons, selections and fp64
// additions a lane and one reduction, five to eight of them a row, where a bitonic sort of the row in registers
// ran 55 stages at EPL = 16.  Sort / this, random keys: 169 / 82 us at 32 x 65536, 32 / 19 at 48 x 17550 (EPL = 8), 35 / 22 at
// 32 x 32768 causal; with all keys equal 145 / 60, half of them 166 / 103 (190 and 178 by halving alone).  Where the launch
// is one wave's latency: EPL = 1 7.8 / 6.8, EPL = 2 11.7 / 12.3, EPL = 4 no difference.
// The ranks cover the n key blocks that the row sees (n <= 64 EPL); the others are 0 in the mask.
// row_at(j): the row's logit of key block j < n; cand: 2 FEW doubles of LDS of this wave's own (may be where row_at reads
// from: all logits are read before the first candidate is written).
constexpr int FEW = 32;
template <int EPL, class RowAt>
__device__ __forceinline__ void topcdf_row(RowAt row_at, const int i, const double sim_q_i, const double* __restrict__ sk,
                                           const Shape& s, const double tau, const double theta, const int causal,
                                           const int n, const int lane, double* cand, uint8_t* __restrict__ out) {
    typedef unsigned long long u64;
    const double NEG = -__builtin_inf();
    if (sim_q_i < theta) {   // a query block that is not self-similar keeps every visible key block
        for (int j = lane; j < s.Tn; j += 64) out[j] = j < n ? 1 : 0;
        return;
    }
    // 1.-2. masked logits, softmax, probabilities (entry e of a lane: key block 64 e + lane)
    double p[EPL];
    unsigned int fix = 0;   // bit e: the key block is not self-similar (kept whatever its rank)
    double mx = NEG;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {   // (loads without conditions: all in flight together)
        const int j = min(64 * e + lane, n - 1);
        p[e] = row_at(j);
        fix |= static_cast<unsigned int>(sk[j] < theta) << e;
    }
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        if (64 * e + lane >= n || (fix >> e & 1)) p[e] = NEG;
        mx = fmax(mx, p[e]);
    }
    mx = wave_max(mx);
    double z = 0.0;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        p[e] = (p[e] == NEG) ? 0.0 : exp(p[e] - mx);
        z += p[e];
    }
    z = group_sum<64>(z);
    // (one division per lane; x * (1 / z) is within two roundings of x / z, far inside the band in which a
    // TopCdf decision counts as undecided)
    const double rz = z > 0.0 ? 1.0 / z : 0.0;
    double tot = 0.0;
    u64 key[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const int j = 64 * e + lane;
        p[e] *= rz;
        tot += p[e];
        key[e] = j < n ? ((static_cast<u64>(__double_as_longlong(p[e])) & ~0xFFFFull) | static_cast<u64>(0xFFFF - j))
                       : 0ull;   // below every key
    }
    tot = uniform_f64(group_sum<64>(tot));
    const double thresh = tau * tot;

    // 3. the bracket
    const auto bits = [](double v) { return static_cast<u64>(__double_as_longlong(v)); };
    u64 lo = 0, hi = (bits(uniform_f64(rz)) | 0xFFFFull) + 1;   // (no probability exceeds exp(0) / z)
    int n_lo = n, n_hi = 0;                                      // entries from lo, from hi on
    double mass_hi = 0.0;                                        // mass from hi on
    u64 mid = bits(uniform_f64((1.0 - tau) * tot * __builtin_amdgcn_rcp(static_cast<double>(n)) * 0.999));
    int idle = 0;          // probes that left no entry out
    bool equal = false;    // the bracket's entries are equal up to their index
#pragma unroll 1
    while (n_lo - n_hi > FEW && hi - lo > 1) {
        if (idle == 2) {   // shrink it to the keys in it
            idle = 0;
            double least = NEG, most = NEG;
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                const bool in = key[e] >= lo && key[e] < hi && key[e] != 0;
                const double k = __longlong_as_double(static_cast<long long>(key[e]));
                least = fmax(least, in ? -k : NEG);
                most = fmax(most, in ? k : NEG);
            }
            least = -uniform_f64(wave_max(least)), most = uniform_f64(wave_max(most));
            if (!(least < most)) break;   // (a row of NaN: no key is in it)
            lo = bits(least), hi = bits(most) + 1;
            equal = ((lo ^ (hi - 1)) >> 16) == 0;
            if (equal) break;
        }
        if (mid <= lo || mid >= hi) mid = lo + (hi - lo) / 2;
        double m = 0.0;
        int c = 0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
            const bool ge = key[e] >= mid;
            m += ge ? p[e] : 0.0;
            c += __popcll(__builtin_amdgcn_ballot_w64(ge));
        }
        m = uniform_f64(group_sum<64>(m));
        idle += c == (m >= thresh ? n_lo : n_hi);
        if (m >= thresh) lo = mid, n_lo = c;
        else hi = mid, n_hi = c, mass_hi = m;
        mid = 0;
    }
    u64 from = hi;            // the cut: entries with keys from here on are kept,
    unsigned int kept_e = 0;  // and (bit e) those of equal ones that rank before it
    if (equal) {
        double each = NEG;
#pragma unroll
        for (int e = 0; e < EPL; ++e) each = fmax(each, key[e] >= lo && key[e] < hi ? p[e] : NEG);
        each = uniform_f64(wave_max(each));
        int before = 0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {   // ascending by index
            const bool in = key[e] >= lo && key[e] < hi;
            const u64 bal = __builtin_amdgcn_ballot_w64(in);
            const int r = before + __popcll(bal & ((1ull << lane) - 1ull));
            kept_e |= static_cast<unsigned int>(in && each > 0.0 && mass_hi + r * each < thresh) << e;
            before += __popcll(bal);
        }
    } else {
        // 4. the entries in it, one per lane: kept iff the mass before them is below the threshold; the smallest kept key is
        // the cut (an entry without mass is never kept)
        int few = 0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
            const bool in = key[e] >= lo && key[e] < hi && key[e] != 0;
            const u64 bal = __builtin_amdgcn_ballot_w64(in);
            if (in) {
                const int at = few + __popcll(bal & ((1ull << lane) - 1ull));
                cand[2 * at] = __longlong_as_double(static_cast<long long>(key[e]));
                cand[2 * at + 1] = p[e];
            }
            few += __popcll(bal);
        }
        __builtin_amdgcn_wave_barrier();   // (written and read by this wave only, whose LDS accesses complete in order)
        static_assert(FEW == 32, "two lanes per candidate, each adds up every other one of those before it");
        const double my_key = cand[2 * (lane & 31)], my_p = cand[2 * (lane & 31) + 1];
        double before = 0.0;
#pragma unroll 8
        for (int c = 0; c < few; c += 2) {
            const double2 x = reinterpret_cast<const double2*>(cand)[c + (lane >> 5)];   // (one behind the last may be read)
            before += c + (lane >> 5) < few && x.x > my_key ? x.y : 0.0;
        }
        before = mass_hi + add_partner<32>(before);
        const bool kept = (lane & 31) < few && my_p > 0.0 && before < thresh;
        // (keys are positive as fp64 numbers and order alike)
        const double cut = -uniform_f64(wave_max(kept ? -my_key : NEG));
        if (cut < -NEG) from = bits(cut);
    }

    // 5. fix-block overrides and causal rules
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const int j = 64 * e + lane;
        const bool m = (key[e] >= from && p[e] > 0.0) || (kept_e >> e & 1) || (fix >> e & 1) || (causal && j == (i * BQ) / BK);
        if (j < s.Tn) out[j] = j < n && m ? 1 : 0;
    }
    for (int j = 64 * EPL + lane; j < s.Tn; j += 64) out[j] = 0;
}
// The same with the fewest entries per lane that hold the row: a causal row of a quarter (half) of the blocks.  Predictor call
// without / with that, causal: 382 / 375 us at 32 x 65536 x 128, 206 / 192 at 8 x 131072 x 64, 78 / 76 at 48 x 17550 x 64.
template <int EPL, class RowAt>
__device__ __forceinline__ void topcdf_row_of(RowAt row_at, const int i, const double sim_q_i, const double* __restrict__ sk,
                                              const Shape& s, const double tau, const double theta, const int causal,
                                              const int lane, double* cand, uint8_t* __restrict__ out) {
    const int n = visible_blocks(s, i, causal);
    if constexpr (EPL >= 8) {
        if (n <= 16 * EPL) {
            topcdf_row<EPL / 4>(row_at, i, sim_q_i, sk, s, tau, theta, causal, n, lane, cand, out);
            return;
        }
    }
    if constexpr (EPL >= 4) {
        if (n <= 32 * EPL) {
            topcdf_row<EPL / 2>(row_at, i, sim_q_i, sk, s, tau, theta, causal, n, lane, cand, out);
            return;
        }
    }
    topcdf_row<EPL>(row_at, i, sim_q_i, sk, s, tau, theta, causal, n, lane, cand, out);
}

// One mask row per wave, the logits from memory.
template <int EPL>
__global__ __launch_bounds__(256) void topcdf_wave_kernel(const double* __restrict__ logits,
                                                           const double* __restrict__ sim_q,
                                                           const double* __restrict__ sim_k, Shape s,
                                                           HeadParams tau_h, HeadParams theta_h, int causal,
                                                           int n_rows, uint8_t* __restrict__ mask) {
    __shared__ __align__(16) double cand[4][2 * FEW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rowid = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x) * 4 + wave);   // (b, h, i) flattened
    if (rowid >= n_rows) return;
    const int i = rowid % s.Tm;
    const long long bh = rowid / s.Tm;
    const int op = s.operand(static_cast<int>(bh));   // (Shape: settings of one launch)
    const int h = s.param(static_cast<int>(bh), static_cast<int>(bh % s.H));
    const long long op_row = (long long)op * s.Tm + i;
    const double* row = logits + op_row * s.Tn;
    topcdf_row_of<EPL>([&](int j) { return row[j]; }, i, sim_q[op_row], sim_k + (long long)op * s.Tn, s, static_cast<double>(tau_h.v[h]),
                    static_cast<double>(theta_h.v[h]), causal, lane, cand[wave],
                    mask + (long long)rowid * s.Tn);
}

// The predictor of short rows in one launch, and beside it the K quantization, which waits for the same block
// statistics: the first n_pred workgroups take R mask rows each (the logits of the 16 x 16 tiles over these rows
// by R waves into LDS, then one row per wave), the others quantize `per_wg` K blocks of one head, with the head's
// token mean of K computed on the spot (in the order k_mean_kernel adds: the same bits).
// What bounds it is latency: the logits' operand loads, one chain of d / 4 fp64 matrix products (140 cycles each while
// one wave has the unit), the softmax's reductions and the probes for the cut, one after the other; logits through
// memory and a launch for each of the four passes came on top of that.  (The logits as fp64 fused multiply-adds, a wave
// per d / 8 channels with the queries in scalar registers: 25.5 against 22.4 us a call at 2 x 2048 x 64, the scalar
// loads wait for each other.)
template <int D, int DT, int EPL, int R>
__global__ __launch_bounds__(64 * R) void predict_quant_kernel(
    const double* __restrict__ pooled_q, const double* __restrict__ ksum_t, const double* __restrict__ sim_q,
    const double* __restrict__ sim_k, const uint16_t* __restrict__ K, Shape s, double sm_scale, HeadParams tau_h,
    HeadParams theta_h, int causal, int n_pred, int per_wg, uint8_t* __restrict__ mask, int8_t* __restrict__ Kq,
    float* __restrict__ k_scale) {
    constexpr int NPAD = 64 * EPL;
    static_assert(R % 4 == 0 && R <= 16, "rows of one 16-row tile, whole groups of 256 threads");
    struct Rows {
        double lg[R][NPAD];       // logits, then a row's candidates
    };
    struct Quant {
        float mean[D];
        float amax[2][R / 4][4];
    };
    __shared__ __align__(16) union {
        Rows rows;
        Quant quant;
    } lds;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    int id = blockIdx.x;
    if (id < n_pred) {
        const int groups = (s.Tm + R - 1) / R;
        const long long bh = id / groups;
        const int i0 = id % groups * R, l16 = lane & 15, kk = lane >> 4;
        const double* qrow = pooled_q + (bh * s.Tm + min(i0 + l16, s.Tm - 1)) * D + kk;   // rows past Tm or R: not used
#pragma unroll 1
        for (int j0 = wave * 16; j0 < visible_blocks(s, i0 + R - 1, causal); j0 += 16 * R) {
            const double* kcol = ksum_t + bh * D * s.Tn + (long long)kk * s.Tn + min(j0 + l16, s.Tn - 1);
            v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < D; c += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qrow[c], kcol[(long long)c * s.Tn], acc, 0, 0, 0);
            const int j = j0 + l16;
            if (j < s.Tn) {
                const double cnt = static_cast<double>(min(BK, s.N - j * BK));
#pragma unroll
                for (int r = 0; r < R / 4; ++r) lds.rows.lg[4 * r + kk][j] = sm_scale * (acc[r] / cnt);
            }
        }
        __syncthreads();
        const int i = i0 + wave, h = static_cast<int>(bh % s.H);
        if (i >= s.Tm) return;
        const double* row = lds.rows.lg[wave];
        topcdf_row_of<EPL>([&](int j) { return row[j]; }, i, sim_q[bh * s.Tm + i], sim_k + bh * s.Tn, s,
                        static_cast<double>(tau_h.v[h]), static_cast<double>(theta_h.v[h]), causal, lane,
                        lds.rows.lg[wave], mask + (bh * s.Tm + i) * s.Tn);
        return;
    }
    id -= n_pred;
    const int wgs = (s.Tn + per_wg - 1) / per_wg;
    const long long bh = id / wgs;
    const int t0 = id % wgs * per_wg;
    // token mean of K: 16 lanes per channel; lane l of them holds the partial sums that lanes l, l + 16, l + 32
    // and l + 48 of k_mean_kernel hold, combined as there
    for (int c = threadIdx.x >> 4; c < D; c += 4 * R) {
        const double* row = ksum_t + (bh * D + c) * s.Tn;
        double v[EPL][4], a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < EPL; ++e)
#pragma unroll
            for (int q = 0; q < 4; ++q)   // (loads without conditions, all in flight: one by one they were a memory latency each)
                v[e][q] = row[min(64 * e + 16 * q + (lane & 15), s.Tn - 1)];
#pragma unroll
        for (int e = 0; e < EPL; ++e)
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] += 64 * e + 16 * q + (lane & 15) < s.Tn ? v[e][q] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = group_sum<16>(a[q]);
        const double sum = (a[0] + a[1]) + (a[2] + a[3]);
        if ((lane & 15) == 0) lds.quant.mean[c] = static_cast<float>(sum / static_cast<double>(s.N));
    }
    __syncthreads();
    const int tid = threadIdx.x & 255, part = threadIdx.x >> 8, cchunk = tid % (D / 8);
    float mean[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) mean[e] = lds.quant.mean[cchunk * 8 + e];
    const uint16_t* base = K + (bh / s.H) * s.sb + (bh % s.H) * s.sh;
    const int t1 = min(t0 + per_wg, s.Tn);
    int turn = 0;   // two sets of block maxima in turn: one barrier per block
    for (int t = t0; t < t1; t += R / 4, turn ^= 1)
        quant_k_block<D, DT>(base, s, bh, t + part < t1 ? t + part : s.Tn, tid, mean, lds.quant.amax[turn][part], Kq, k_scale);
}

// The mask as an index list: one wave per mask row compacts the kept block indices with ballots, 64 entries
// at a time, in ascending order; the rest of the row is -1.  Eight ballots' entries are loaded before the first of them
// is needed: with a load per ballot a row was a chain of T_n / 64 memory latencies (15.7 against 20.5 us at 32 heads of
// 512 x 1024 blocks, 15.3 against 21.9 us at 8 heads of 1024 x 2048).
__global__ __launch_bounds__(256) void mask_lut_kernel(const uint8_t* __restrict__ mask, int Tn, int n_rows,
                                                       int32_t* __restrict__ lut, int32_t* __restrict__ lut_count) {
    constexpr int AHEAD = 8;
    const int row = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= n_rows) return;
    const uint8_t* m = mask + static_cast<long long>(row) * Tn;
    int32_t* out = lut + static_cast<long long>(row) * Tn;
    int n = 0;
    for (int base = 0; base < Tn; base += 64 * AHEAD) {
        uint8_t keep[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            const int j = base + 64 * q + lane;
            keep[q] = j < Tn ? m[j] : 0;
        }
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            const unsigned long long bal = __ballot(keep[q] != 0);
            if (keep[q] != 0) out[n + __popcll(bal & ((1ull << lane) - 1ull))] = base + 64 * q + lane;
            n += __popcll(bal);
        }
    }
    for (int j = n + lane; j < Tn; j += 64) out[j] = -1;
    if (lane == 0) lut_count[row] = n;
}

}  // namespace

hipError_t launch_mask_lut(const uint8_t* mask, const Shape& s, int32_t* lut, int32_t* lut_count, hipStream_t st) {
    const int n_rows = s.B * s.H * s.Tm;
    hipLaunchKernelGGL(mask_lut_kernel, dim3((n_rows + 3) / 4), dim3(256), 0, st, mask, s.Tn, n_rows, lut, lut_count);
    return hipGetLastError();
}

hipError_t launch_logits(const double* pooled_q, const double* ksum_t, const Shape& s, float sm_scale, int causal,
                         double* logits, hipStream_t st) {
    // two row tiles of 16 pooled queries per wave where there are enough rows to fill the chip that way
    // (measured: 55 against 61 us at T_m = 360, 33 against 39 us at T_m = 256 with 32 heads; 18 against 17 us at T_m = 138)
    const int rt = s.Tm >= 192 ? 2 : 1;
    dim3 grid((s.Tn + 63) / 64, (s.Tm + 64 * rt - 1) / (64 * rt), s.B * s.H);
    const double scale = sm_scale > 0.f ? static_cast<double>(sm_scale) : 1.0 / sqrt(static_cast<double>(s.d));
#define CALL(D, RT) hipLaunchKernelGGL((logits_kernel<D, RT>), grid, dim3(256), 0, st, pooled_q, ksum_t, s, scale, causal, logits)
    if (s.d == 64) { if (rt == 2) CALL(64, 2); else CALL(64, 1); }
    else { if (rt == 2) CALL(128, 2); else CALL(128, 1); }
#undef CALL
    return hipGetLastError();
}

hipError_t launch_topcdf(const double* logits, const double* sim_q, const double* sim_k, const Shape& s,
                         const HeadParams& tau, const HeadParams& theta, int causal, uint8_t* mask,
                         hipStream_t st) {
    const int n_rows = s.B * s.H * s.Tm;
#define CALLW(EPL)                                                                                                 \
    hipLaunchKernelGGL((topcdf_wave_kernel<EPL>), dim3((n_rows + 3) / 4), dim3(256), 0, st, logits, sim_q, sim_k, s, \
                       tau, theta, causal, n_rows, mask)
    if (s.Tn <= 256) { CALLW(4); return hipGetLastError(); }
    if (s.Tn <= 512) { CALLW(8); return hipGetLastError(); }
    if (s.Tn <= 1024) { CALLW(16); return hipGetLastError(); }
    if (s.Tn <= 2048) { CALLW(32); return hipGetLastError(); }
#undef CALLW
    // longer rows: one workgroup per row, sorted in LDS
    int npad = 2;
    while (npad < s.Tn) npad <<= 1;
    const size_t smem = static_cast<size_t>(npad) * (sizeof(double) + sizeof(unsigned long long) + 1);
    // 68 KB at the longest rows: more than the 64 KB a launch gets without asking (the CU has 160 KB)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(topcdf_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem));
    if (e != hipSuccess) return e;
    dim3 grid(s.Tm, s.H, s.B);
    hipLaunchKernelGGL(topcdf_kernel, grid, dim3(256), smem, st, logits, sim_q, sim_k, s, tau, theta, causal,
                       npad, mask);
    return hipGetLastError();
}

hipError_t launch_predict_quant(const double* pooled_q, const double* ksum_t, const double* sim_q, const double* sim_k,
                                const void* K, const Shape& s, const HeadParams& tau, const HeadParams& theta,
                                float sm_scale, int causal, uint8_t* mask, int8_t* Kq, float* k_scale, hipStream_t st) {
    if (!short_call(s)) return hipErrorInvalidValue;
    constexpr int R = 8;   // 4 and 16 rows per workgroup: within 3 % of it, either side (33.4 / 31.6 / 31.3 us a call at
                         // 2 x 2048 x 64 with 16 / 8 / 4, 168 / 168 / 170 us at 24 x 4173 x 128)
    const int BH = s.B * s.H, n_pred = BH * ((s.Tm + R - 1) / R);
    // K blocks per workgroup: enough that reading the block sums for the mean (8 d T_n bytes) stays below reading
    // the blocks themselves (128 d bytes each)
    int per_wg = (s.Tn + 15) / 16;
    per_wg = (per_wg + R / 4 - 1) / (R / 4) * (R / 4);
    const int n_quant = Kq ? BH * ((s.Tn + per_wg - 1) / per_wg) : 0;
    const double scale = sm_scale > 0.f ? static_cast<double>(sm_scale) : 1.0 / sqrt(static_cast<double>(s.d));
    const uint16_t* X = static_cast<const uint16_t*>(K);
#define CALLE(D, DT, EPL)                                                                                          \
    hipLaunchKernelGGL((predict_quant_kernel<D, DT, EPL, R>), dim3(n_pred + n_quant), dim3(64 * R), 0, st, pooled_q, \
                       ksum_t, sim_q, sim_k, X, s, scale, tau, theta, causal, n_pred, per_wg, mask, Kq, k_scale)
#define CALL(D, DT) { if (s.Tn <= 128) CALLE(D, DT, 2); else CALLE(D, DT, 4); }
    if (s.d == 64 && s.dtype == SPARGE_F16) CALL(64, SPARGE_F16)
    else if (s.d == 64 && s.dtype == SPARGE_BF16) CALL(64, SPARGE_BF16)
    else if (s.d == 128 && s.dtype == SPARGE_F16) CALL(128, SPARGE_F16)
    else if (s.d == 128 && s.dtype == SPARGE_BF16) CALL(128, SPARGE_BF16)
    else return hipErrorInvalidValue;
#undef CALL
#undef CALLE
    return hipGetLastError();
}

}  // namespace sparge
