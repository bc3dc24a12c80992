// The sparse flash loop (Alg. 1 lines 7-20) for calls with few Q blocks: one 32-row group per workgroup, its key blocks
// shared out over the waves.
//
// What bounds such calls is latency: attn.hip gives a row group to one wave, which walks its tiles one after the other
// at 0.55 (d = 64) or 0.69 us (d = 128) a tile however empty the chip is.  Here a round takes tiles 4r .. 4r + 3 of the
// group's list; four waves make their scores and P~, four more (d = 64: two) multiply with V:
//   softmax wave w                                             product wave (32 channels)
//   scores of tile 4r + w and their row maxima                 O += P~ V of round r - 1, tile by tile
//   ---- barrier A: the row maxima of the four tiles are exchanged
//   running maximum and moves of the reference maximum         the same, and the stage-2 decisions;
//   through the four tiles in order; P~ of its tile against    V of round r into registers
//   the reference its place in the order gives
//   ---- barrier B: P~ is exchanged; the row sums go from softmax wave to softmax wave
// K_hat and V are copied to LDS a round or two ahead, at d = 64 by two waves that do nothing else; LDS has no room for that
// at d = 128, where the product waves copy beside their products.  A round takes 1.10 us at d = 64 and 1.72 us at d = 128
// (2.3 and 3.0 us for its tiles one after the other in attn.hip; FP8 P~V 1.04 and 1.35, 16-bit Q K^T 1.21 and 2.78 us), bound
// by the softmax waves' instructions (2200 of 2600 cycles) and, at d = 128, by the copies' 96 KB through the unit's 64 bytes a
// cycle.  (With a sum per tile for l, added up by the product waves, 1.02 and 1.91 us, but l in another order.)  On the way: operands loaded from
// memory straight into registers, 2.0 / 3.5 us (32 rows of 32 bytes a load); one kind of wave for everything, 1.5 / 2.4
// us; V copied between the products at d = 64 too, 1.22 us.
// Everything that is decided or rounded per tile is decided and rounded as in attn.hip, and every sum has its order (P~ V:
// tiles in list order on the same matrix instruction; l: one P~ after the other through all tiles), so the two kernels
// give the same bits, infinities and NaN included (of a NaN: that it is one), and the choice between them is one of speed alone (attn_split_pays).
#include "attn_ops.hpp"

namespace sparge {

namespace {

constexpr int SPLIT_WAVES = 4;   // softmax waves, and as many others: d / 32 product waves, the rest copies tiles

struct SplitArgs {
    const void* Qp;
    const void* Kp;
    const float* q_scale;
    const float* k_scale;
    const unsigned char* v_tiles;
    const float* v_scale;
    uint16_t* O;
    const uint8_t* mask;
    unsigned long long* stats;
    Shape s;
    float sm_scale;
    int per_xcd;
    HeadParams lambda_h;
};

// LDS traffic of this wave done, then the barrier: copies from memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// max without the quieting of signalling NaNs that fmaxf costs an instruction per operand for (no operand comes from a
// matrix instruction or v_exp, whose results the assembler would not wait for)
__device__ __forceinline__ float vmax(float x, float y) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

// two fp32 -> a pair of 16-bit values in one register, round to nearest even
template <int DT>
__device__ __forceinline__ int pack2(float x, float y) {
    const v2f v = {x, y};
    if constexpr (DT == SPARGE_BF16) return __builtin_bit_cast(int, __builtin_convertvector(v, v2bf));
    else return __builtin_bit_cast(int, __builtin_convertvector(v, v2h));
}

template <int D, int DT, bool CAUSAL, bool FP8, bool QK16>
__global__ __launch_bounds__(128 * SPLIT_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_split_kernel(const SplitArgs a) {
    constexpr int NW = SPLIT_WAVES;
    constexpr int NSTEP = QK16 ? D / 16 : D / 32;  // MFMA steps along d
    constexpr int NDT = D / 32;                    // 32-channel output tiles, one per wave
    constexpr int NV = FP8 ? 2 : 4;                // 16-byte operand pieces of a tile's 32 channels; of its P~
    constexpr int V_BYTES = D * BK * (FP8 ? 1 : 2);
    constexpr int K_ROWB = QK16 ? 2 * D : D, K_CPR = K_ROWB / 16;   // bytes, 16-byte chunks of a K row in LDS
    constexpr int K_DMA = BK * K_ROWB / 1024, VT_DMA = NV;   // wave-wide copies of a K tile; of a V tile's 32 channels
    constexpr float SLACK = FP8 ? SPARGE_REF_SLACK_LOG2_FP8 : SPARGE_REF_SLACK_LOG2;
    constexpr float BIAS = QK16 ? 0.f : MAGIC_F;
    const float NEG = -__builtin_inff();
    constexpr int KB = QK16 && D == 128 ? 1 : 2;   // K_hat buffers: rounds ahead (LDS holds no second one there)
    __shared__ __align__(1024) unsigned char Ks[KB][NW][K_DMA * 1024];
    constexpr int VB = D == 64 ? 2 : 1;            // V buffers
    __shared__ __align__(1024) unsigned char Vs[VB][NDT][NW][VT_DMA * 1024];   // a product wave's channels of the four tiles
    __shared__ __align__(16) v4i ps[NW][NV][64];   // P~ of the round's tiles as the P~V operand
    __shared__ __align__(16) float row_max[RG][NW];
    __shared__ __align__(8) unsigned long long row_sums[64];   // per lane of the scores: l so far, tiles in it
    volatile __attribute__((address_space(3))) unsigned long long* const row_sum =
        (volatile __attribute__((address_space(3))) unsigned long long*)row_sums + (threadIdx.x & 63);
    __shared__ float scl[SPLIT_MAX_TN + 4 * NW];   // per kept tile: q_scale * k_scale * sm_scale * log2(e)
    __shared__ __align__(8) uint16_t jl[SPLIT_MAX_TN + 4 * NW];   // kept key blocks of this row, ascending; then zeros

    const Shape& s = a.s;
    // the arguments in one round trip (left to themselves the loads of an argument wait for its first use, one after the other)
    asm volatile("" ::"s"(a.Qp), "s"(a.Kp), "s"(a.q_scale), "s"(a.k_scale), "s"(a.v_tiles), "s"(a.mask), "s"(a.stats), "s"(a.per_xcd),
                 "s"(a.sm_scale), "s"(s.H), "s"(s.N), "s"(s.Tm), "s"(s.Tn), "s"(s.op_bh), "s"(s.dense_bh), "s"(s.by_setting), "s"(s.one_mask));
    const int n_rg = (s.N + RG - 1) / RG;
    // consecutive workgroups land on different XCDs: each XCD takes a contiguous range of row groups, so that its L2
    // serves few heads; causal heads start with their longest rows
    const int work = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
    if (work >= s.B * s.H * n_rg) return;
    const int bh = work / n_rg;
    const int g = CAUSAL ? n_rg - 1 - work % n_rg : work % n_rg;
    const int b = bh / s.H, h = bh % s.H, i = g / (BQ / RG);
    const int op = s.operand(bh), own = bh - s.dense_bh;   // (Shape: settings of one launch)
    const int lane = threadIdx.x & 63, l32 = lane & 31, hl = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int qrow = g * RG + l32;
    const bool row_counts = qrow < s.N;

    const float lam2 = a.lambda_h.v[s.param(own, h)] * LOG2E;
    v4i qf[NSTEP];
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
        qf[st] = v4i{0, 0, 0, 0};
        if (wave < NW && row_counts)
            qf[st] = QK16 ? *reinterpret_cast<const v4i*>(static_cast<const uint16_t*>(a.Qp) + b * s.sb + h * s.sh +
                                                          (long long)qrow * s.sn + st * 16 + hl * 8)
                          : *reinterpret_cast<const v4i*>(static_cast<const int8_t*>(a.Qp) +
                                                          ((long long)op * s.N + qrow) * D + st * 32 + hl * 16);
    }
    // ---- the Q block's kept key blocks in ascending order: every wave counts all of them, the first two write a half.
    // A causal group runs only the tiles it sees (the other ones of its block change nothing).
    const int jmax = CAUSAL ? min(s.Tn, (i * BQ + BQ - 1) / BK + 1) : s.Tn;
    const int jvis = CAUSAL ? min(jmax, (g * RG + RG - 1) / BK + 1) : jmax;
    // (the loop of attn.hip takes key blocks from j_rag on, and the one before them, with element masks)
    const int j_rag = CAUSAL ? min(s.N / BK, 2 * i) : s.N / BK;
    int listed = 0, cnt = 0, full = 0;   // kept blocks of the Q block; those that this group sees; those before j_rag
    {
        constexpr int NL = SPLIT_MAX_TN / 64;   // flags a lane
        static_assert(NL == 2 && SPLIT_MAX_TN == 64 * NL, "two loads in one block below");
        // (loads without conditions and in one block, all in flight together; without a mask they read what they like)
        const bool dense = !a.mask || own < 0;
        const uint8_t* mrow = dense ? a.v_tiles : a.mask + ((long long)(s.one_mask ? op : own) * s.Tm + i) * s.Tn;
        unsigned int mk[NL];
#pragma unroll
        for (int q = 0; q < NL; ++q) mk[q] = mrow[min(q * 64 + lane, jmax - 1)];
        const float sc = QK16 ? 1.f : a.k_scale[(long long)op * s.Tn + min((wave & (NL - 1)) * 64 + lane, jmax - 1)];
        const float qs = (QK16 ? 1.f : a.q_scale[(long long)op * s.Tm + i]) * a.sm_scale * LOG2E;
        asm volatile("" ::"v"(mk[0]), "v"(mk[1]), "v"(sc), "v"(qs), "v"(lam2));
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int j = q * 64 + lane;
            const bool keep = (dense || mk[q] != 0) && j < jmax;
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(keep);
            if (q == wave && keep) {
                const int pos = listed + __popcll(bal & ((1ull << lane) - 1ull));
                jl[pos] = static_cast<uint16_t>(j);
                scl[pos] = fmaxf(qs * sc, 1e-30f);   // never 0: a masked score is -inf * scale
            }
            listed += __popcll(bal);
            cnt += __popcll(__builtin_amdgcn_ballot_w64(keep && j < jvis));
            full += __popcll(__builtin_amdgcn_ballot_w64(keep && j < j_rag));
        }
    }
    if (wave == NW && lane < 4 * NW) jl[listed + lane] = 0;   // copies behind the list fetch a tile nobody reads
    if (wave == NW) *row_sum = 0ull;
    lds_barrier();

    float m_true = NEG, m_ref = NEG;
    // what both kinds of waves follow: the running maximum through the round's tiles (ml: their row maxima) ...
    float ml[NW], m[NW];
    auto follow = [&](int t0) -> bool {   // -> does the reference maximum move somewhere in this round?
        const float4 ml4 = *reinterpret_cast<const float4*>(row_max[l32]);
        ml[0] = ml4.x, ml[1] = ml4.y, ml[2] = ml4.z, ml[3] = ml4.w;
#pragma unroll
        for (int w = 0; w < NW; ++w) m[w] = vmax(w ? m[w - 1] : m_true, ml[w]);
        m_true = m[NW - 1];
        asm("" : "+s"(t0));   // (the first round is not worth a copy of the loop of its own)
        if (t0 == 0) m_ref = ml[0];
        return __builtin_amdgcn_ballot_w64(row_counts && m[NW - 1] - m_ref > SLACK) != 0;   // the maximum only grows
    };
    // ... and whether the reference moves to it at tile w (then O and l are multiplied by f)
    auto moves = [&](int w, float& f) -> bool {
        if (__builtin_amdgcn_ballot_w64(row_counts && m[w] - m_ref > SLACK) == 0) return false;
        f = __builtin_amdgcn_exp2f(m_ref - m[w]);
        m_ref = m[w];
        return true;
    };

    if (wave < NW) {
        v16i magic;   // start of the scores (opaque: it stays in registers)
#pragma unroll
        for (int r = 0; r < 16; ++r) magic[r] = QK16 ? 0 : MAGIC_I;
        asm volatile("" : "+v"(magic));
        int buf = 0;
        int j = jl[wave];
        float sc = scl[wave];
        // l takes one P~ after the other, tile by tile: it goes from wave to wave, and a wave waits until it holds the tiles
        // before its own.  Wave 0 adds its tile at the end of the round; waves 1, 2 and 3 add theirs in the next round, beside
        // the scores, before barrier A and behind it: each after the one it waits for, which in that interval between two
        // barriers waits for nobody itself, so every wait ends and is nearly always over before it begins.
        float p[32];
        float f_own = 1.f;   // the move of the reference maximum at the own tile
        auto add_tile = [&](int t) {
#pragma clang fp contract(off)   // (the move and the first addition round one after the other)
            unsigned long long sum_n;
            do sum_n = *row_sum;
            while (__builtin_amdgcn_ballot_w64(static_cast<int>(sum_n >> 32) != t) != 0);
            float l = __uint_as_float(static_cast<uint32_t>(sum_n)) * f_own;
#pragma unroll
            for (int e = 0; e < 32; ++e) l += p[e];
            *row_sum = static_cast<unsigned long long>(static_cast<uint32_t>(t + 1)) << 32 | __float_as_uint(l);
        };
        if (cnt > 0) lds_barrier();   // K_hat of the first round is there
        for (int t0 = 0; t0 < cnt; t0 += NW) {
            const bool live = t0 + wave < cnt;   // there is a tile for this wave
            const int j_next = jl[t0 + NW + wave];
            const float sc_next = scl[t0 + NW + wave];
            float m_loc = NEG;
            v16i S[2];
            if (live) {
                const unsigned char* const Kw = Ks[buf][wave];
#pragma unroll
                for (int st = 0; st < NSTEP; ++st) {
#pragma unroll
                    for (int kh = 0; kh < 2; ++kh) {
                        const v4i kf = *reinterpret_cast<const v4i*>(Kw + (kh * 32 + l32) * K_ROWB + (((st * 2 + hl) ^ swz<K_ROWB>(l32)) * 16));
                        const v16i c = st == 0 ? magic : S[kh];
                        if constexpr (QK16) S[kh] = __builtin_bit_cast(v16i, mfma16<DT>(kf, qf[st], __builtin_bit_cast(v16f, c)));
                        else S[kh] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf, qf[st], c, 0, 0, 0);
                    }
                }
                if (wave == 1 && t0 > 0) add_tile(t0 - NW + 1);   // (the scores are not there yet)
                // biased integers compare like the scores (-inf is a negative integer)
                const int ju = __builtin_amdgcn_readfirstlane(j);
                if (ju * BK + BK > s.N || (CAUSAL && ju * BK + BK - 1 > g * RG)) {
                    const int key_lim = (CAUSAL ? min(s.N - 1, qrow) : s.N - 1) - ju * BK - 4 * hl;
#pragma unroll
                    for (int e = 0; e < 32; ++e) {
                        const int r = e & 15;
                        if ((e >> 4) * 32 + 8 * (r >> 2) + (r & 3) > key_lim) S[e >> 4][r] = __float_as_int(NEG);
                    }
                }
                if constexpr (QK16) {
                    float m0 = __int_as_float(S[0][0]), m1 = __int_as_float(S[1][0]);
#pragma unroll
                    for (int r = 1; r < 16; ++r) {
                        m0 = fmaxf(m0, __int_as_float(S[0][r]));
                        m1 = fmaxf(m1, __int_as_float(S[1][r]));
                    }
                    m_loc = fmaxf(m0, m1) * sc;
                } else {
                    int m0 = S[0][0], m1 = S[1][0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) {
                        m0 = max(m0, S[0][r]);
                        m1 = max(m1, S[1][r]);
                    }
                    m_loc = (__int_as_float(max(m0, m1)) - BIAS) * sc;
                }
                m_loc = max_across_halves(m_loc);
                if (t0 + wave == 0) m_loc = fmaxf(m_loc, NEG);   // (scores that are all NaN: the running maximum starts at -inf)
            }
            if (!live && wave == 1 && t0 > 0) add_tile(t0 - NW + 1);
            if (hl == 0) row_max[l32][wave] = m_loc;
            if (wave == 2 && t0 > 0) add_tile(t0 - NW + 2);
            lds_barrier();   // A
            if (wave == 3 && t0 > 0) add_tile(t0 - NW + 3);
            const bool any_move = follow(t0);
            float ref_own = m_ref;
            f_own = 1.f;
            if (any_move) {
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    float f;
                    const bool moved = moves(w, f);
                    if (w == wave) {
                        ref_own = m_ref;
                        if (moved) f_own = f;
                    }
                }
            }
            if (live) {
                float cx = __builtin_fmaf(-BIAS, sc, -ref_own);
                if constexpr (FP8) cx += 6.807354927062988f;   // P~ scaled by 448 / 2^2: log2(448) - 2
                // a row that has seen no key yet: its masked scores are all -inf (and scores of -inf themselves give NaN)
                if (ref_own == NEG && t0 + wave + 1 >= full) cx = 0.f;
#pragma unroll
                for (int e = 0; e < 32; ++e)
                    p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(__int_as_float(S[e >> 4][e & 15]), sc, cx));
                int pk[NV * 4];
                if constexpr (FP8) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        pk[q] = __builtin_amdgcn_cvt_pk_fp8_f32(p[4 * q], p[4 * q + 1], 0, false);
                        pk[q] = __builtin_amdgcn_cvt_pk_fp8_f32(p[4 * q + 2], p[4 * q + 3], pk[q], true);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 16; ++q) pk[q] = pack2<DT>(p[2 * q], p[2 * q + 1]);
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) ps[wave][q][lane] = v4i{pk[4 * q], pk[4 * q + 1], pk[4 * q + 2], pk[4 * q + 3]};
                if (wave == 0) add_tile(t0);
            }
            lds_barrier();   // B
            j = j_next;
            sc = sc_next;
            if (KB == 2) buf ^= 1;
        }
        if (cnt > 0) {
            const int t = (cnt - 1) / NW * NW + wave;
            if (wave > 0 && t < cnt) add_tile(t);
            lds_barrier();   // l is there
        }
        if (a.stats && own >= 0 && threadIdx.x == 0) {   // row groups whose last row sees the key block; tiles once per Q block
            unsigned long long* st = a.stats + own * 4;
            atomicAdd(&st[3], (unsigned long long)(CAUSAL ? min(jmax, (min(g * RG + RG, s.N) - 1) / BK + 1) : jmax));
            if (g % (BQ / RG) == 0) {
                atomicAdd(&st[0], (unsigned long long)listed);
                atomicAdd(&st[2], (unsigned long long)jmax);
            }
        }
        return;
    }

    // ---- copies: d = 64: by two waves of their own, two tiles of a round each; d = 128: by the four product waves
    const int hw = wave - NW;
    constexpr int K_TILES = D == 128 ? 1 : 2;
    const int k_tile0 = D == 128 ? hw : 2 * (hw - NDT);
    const unsigned char* kbase = static_cast<const unsigned char*>(a.Kp) +
                                 (QK16 ? 2 * (b * s.sb + h * s.sh) : (long long)op * s.N * D);
    const int k_rowg = QK16 ? static_cast<int>(2 * s.sn) : D;  // bytes between K rows in memory
    // 16-byte chunks are XOR-ed on the memory side of a copy as the operand reads expect
    const int k_row = lane / K_CPR, k_phys = lane % K_CPR;
    auto copy_k = [&](int t0, int buf) {   // rows past N repeat the last one (they are masked)
#pragma unroll
        for (int k = 0; k < K_TILES; ++k) {
            const int j = __builtin_amdgcn_readfirstlane(static_cast<int>(jl[t0 + k_tile0 + k]));
            const uint32_t dst = lds_address(Ks[0][k_tile0 + k]) + buf * (NW * K_DMA * 1024);
            const unsigned char* src = kbase + (long long)j * BK * k_rowg;
            const int last = s.N - 1 - j * BK;
            if (last >= BK - 1) {
#pragma unroll
                for (int n = 0; n < K_DMA; ++n) {
                    const int row = n * (64 / K_CPR) + k_row;
                    dma16_at(src, row * k_rowg + ((k_phys ^ swz<K_ROWB>(row)) * 16), dst, n * 1024);
                }
            } else {
#pragma unroll
                for (int n = 0; n < K_DMA; ++n) {
                    const int row = n * (64 / K_CPR) + k_row;
                    dma16_at(src, min(row, last) * k_rowg + ((k_phys ^ swz<K_ROWB>(row)) * 16), dst, n * 1024);
                }
            }
        }
    };
    // ---- copies of V, by the tile's 32-channel parts: d = 64: the copying waves again, both parts of two tiles each; d = 128:
    // a product wave its own part of all four
    uint32_t v_src[VT_DMA];
#pragma unroll
    for (int n = 0; n < VT_DMA; ++n) {
        const int row = n * 8 + lane / 8;
        v_src[n] = FP8 ? n * 1024 + lane * 16 : row * 128 + (((lane % 8) ^ swz<128>(row)) * 16);
    }
    const unsigned char* vbase = a.v_tiles + (long long)op * s.Tn * V_BYTES;
    if (D == 64 && hw >= NDT) {
        auto copy_v = [&](int t0, int buf) {
#pragma unroll
            for (int k = 0; k < K_TILES; ++k) {
                const int j = __builtin_amdgcn_readfirstlane(static_cast<int>(jl[t0 + k_tile0 + k]));
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const uint32_t dst = lds_address(Vs[0][dt][k_tile0 + k]) + buf * (NDT * NW * VT_DMA * 1024);
#pragma unroll
                    for (int n = 0; n < VT_DMA; ++n)
                        dma16_at(vbase + (long long)j * V_BYTES + dt * (VT_DMA * 1024), v_src[n], dst, n * 1024);
                }
            }
        };
        constexpr int KC = K_TILES * K_DMA, VC = K_TILES * NDT * VT_DMA;   // copies of a wave per round
        if (cnt == 0) return;
        copy_k(0, 0);
        copy_v(0, 0);
        if (NW < cnt) {
            copy_k(NW, 1);
            copy_v(NW, 1);
            dma_wait<KC + 2 * VC>();   // K_hat of the first round has landed
        } else {
            dma_wait<VC>();
        }
        lds_barrier();
        int buf = 0;
        // in flight at the top of a round, oldest first: its V, K_hat and V of the next round
        for (int t0 = 0; t0 < cnt; t0 += NW, buf ^= 1) {
            const bool next = t0 + NW < cnt, more = t0 + 2 * NW < cnt;
            if (next) dma_wait<KC + VC>();   // this round's V
            else dma_wait<0>();
            lds_barrier();   // A: the round's scores are made, its K_hat is free
            if (more) copy_k(t0 + 2 * NW, buf);
            if (more) dma_wait<VC + KC>();   // K_hat of the next round
            else if (next) dma_wait<VC>();
            lds_barrier();   // B: the round's V is in registers
            if (more) copy_v(t0 + 2 * NW, buf);
        }
        lds_barrier();
        return;
    }

    // ---- product waves
    const uint32_t v_lds = lds_address(Vs[0][hw][0]);
    vbase += hw * (VT_DMA * 1024);
    int vj[NW];   // key blocks of the V tiles that are copied next
    auto list_v = [&](int t0) {
        const uint2 four = *reinterpret_cast<const uint2*>(&jl[t0]);
        const int lo = __builtin_amdgcn_readfirstlane(four.x), hi = __builtin_amdgcn_readfirstlane(four.y);
        vj[0] = lo & 0xffff, vj[1] = static_cast<unsigned>(lo) >> 16, vj[2] = hi & 0xffff, vj[3] = static_cast<unsigned>(hi) >> 16;
    };
    auto copy_v = [&](int w, int n) { dma16_at(vbase + (long long)vj[w] * V_BYTES, v_src[n], v_lds, (w * VT_DMA + n) * 1024); };
    v16f O;
#pragma unroll
    for (int r = 0; r < 16; ++r) O[r] = 0.f;
    int pv_done = 0;
    if (cnt > 0) {
        if constexpr (D == 128) {
            copy_k(0, 0);
            list_v(0);
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int n = 0; n < VT_DMA; ++n) copy_v(w, n);
            if (KB == 2 && NW < cnt) copy_k(NW, 1);
            // K_hat of the first round has landed
            if (KB == 2 && NW < cnt) dma_wait<K_DMA + NW * VT_DMA>();
            else dma_wait<NW * VT_DMA>();
        }
        lds_barrier();
    }
    int buf = 0;
    for (int t0 = 0; t0 < cnt; t0 += NW) {
        const bool more = t0 + NW < cnt;
        if constexpr (D == 128) {
            list_v(t0 + NW);
            dma_wait<0>();   // this round's V; K_hat of the next one
        }
        lds_barrier();   // A
        const bool any_move = follow(t0);
        v4i vf[NW][NV];
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int p = 0; p < NV; ++p)
                vf[w][p] = *reinterpret_cast<const v4i*>(&Vs[VB == 2 ? buf : 0][hw][w][0] + (FP8 ? p * 1024 + lane * 16 : l32 * 128 + (((p * 2 + hl) ^ swz<128>(l32)) * 16)));
        // stage-2 decisions (Alg. 1 line 15); a tile that is not there has -inf and is not executed
        int votes = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            votes |= (__builtin_amdgcn_ballot_w64(row_counts && ml[w] - m[w] > lam2) != 0) << w;
        if (t0 == 0) votes |= __builtin_amdgcn_ballot_w64(row_counts && ml[0] != NEG) != 0;   // (+inf among them)
        float f[NW];
        int moved = 0;
        if (any_move) {
#pragma unroll
            for (int w = 0; w < NW; ++w) moved |= moves(w, f[w]) << w;
        }
        pv_done += __builtin_popcount(votes);
        // V of the next round takes the place of this one's, half of it here and half beside the products
        if (D == 128 && more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int w = 0; w < NW / 2; ++w)
#pragma unroll
                for (int n = 0; n < VT_DMA; ++n) copy_v(w, n);
        }
        if (D == 128) {
            if (t0 + KB * NW < cnt) copy_k(t0 + KB * NW, buf);
            if (KB == 1) dma_wait<0>();
        }
        buf ^= KB == 2;
        lds_barrier();   // B
        // ---- O of the own channels, tile by tile
        v4i pf[NW][NV];
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int p = 0; p < NV; ++p) pf[w][p] = ps[w][p][lane];
        auto pv = [&](int w) {
            if constexpr (FP8) {
                O = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                    __builtin_shufflevector(vf[w][0], vf[w][1], 0, 1, 2, 3, 4, 5, 6, 7),
                    __builtin_shufflevector(pf[w][0], pf[w][1], 0, 1, 2, 3, 4, 5, 6, 7), O, 0, 0, 0, 0, 0, 0);
            } else {
#pragma unroll
                for (int p = 0; p < NV; ++p) O = mfma16<DT>(vf[w][p], pf[w][p], O);
            }
        };
        const bool copies = D == 128 && more;
        if (votes == 15 && !moved && (D == 64 || more)) {   // the usual round, without branches
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                pv(w);
                if constexpr (D == 128)
#pragma unroll
                    for (int n = 0; n < VT_DMA / 2; ++n) copy_v(NW / 2 + w / 2, (w & 1) * (VT_DMA / 2) + n);
            }
        } else {
            if (copies) {
#pragma unroll
                for (int w = NW / 2; w < NW; ++w)
#pragma unroll
                    for (int n = 0; n < VT_DMA; ++n) copy_v(w, n);
            }
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (t0 + w >= cnt) break;
                if (moved >> w & 1) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) O[r] *= f[w];
                }
                if (votes >> w & 1) pv(w);
            }
        }
    }

    if (cnt > 0) lds_barrier();   // l is there
    const float l = __uint_as_float(static_cast<uint32_t>(*row_sum));
    // ---- O_i = diag(l)^-1 O_i; a lane holds 4 consecutive channels per accumulator quad
    if (row_counts) {
        const float l_tot = sum_across_halves(l);
        const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
        uint16_t* orow = a.O + b * s.sb + h * s.sh + (long long)qrow * s.sn;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int c0 = hw * 32 + 8 * q4 + 4 * hl;
            float4 dv = make_float4(1.f, 1.f, 1.f, 1.f);  // FP8: the channels' V scales
            if (FP8) dv = *reinterpret_cast<const float4*>(a.v_scale + (long long)op * D + c0);
            const float dvs[4] = {dv.x, dv.y, dv.z, dv.w};
            uint16_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = cvt_to16<DT>(O[4 * q4 + e] * inv * dvs[e]);
            uint2 wd;
            wd.x = o[0] | (static_cast<uint32_t>(o[1]) << 16);
            wd.y = o[2] | (static_cast<uint32_t>(o[3]) << 16);
            *reinterpret_cast<uint2*>(orow + c0) = wd;
        }
    }
    if (a.stats && own >= 0 && hw == 0 && lane == 0 && pv_done) atomicAdd(&a.stats[own * 4 + 1], (unsigned long long)pv_done);
}

}  // namespace

hipError_t launch_attn_split(const void* Qp, const void* Kp, const float* q_scale, const float* k_scale,
                             const void* v_tiles, const float* v_scale, const Shape& s, const uint8_t* mask,
                             const HeadParams& lambda, float scale, int causal, void* O, unsigned long long* stats,
                             hipStream_t st) {
    SplitArgs a;
    a.Qp = Qp, a.Kp = Kp, a.q_scale = q_scale, a.k_scale = k_scale;
    a.v_tiles = static_cast<const unsigned char*>(v_tiles), a.v_scale = v_scale;
    a.O = static_cast<uint16_t*>(O), a.mask = mask, a.stats = stats, a.s = s, a.sm_scale = scale, a.lambda_h = lambda;
    a.per_xcd = (s.B * s.H * ((s.N + RG - 1) / RG) + 7) / 8;
    const dim3 grid(a.per_xcd * 8), block(128 * SPLIT_WAVES);
#define CALL3(D, DT, CAUSAL, FP8, QK16) hipLaunchKernelGGL((attn_split_kernel<D, DT, CAUSAL, FP8, QK16>), grid, block, 0, st, a)
#define CALL2(D, DT, FP8, QK16) { if (causal) CALL3(D, DT, true, FP8, QK16); else CALL3(D, DT, false, FP8, QK16); }
#define CALL(D, DT)                                  \
    {                                                \
        if (s.pv_fp8) CALL2(D, DT, true, false)      \
        else if (s.qk16) CALL2(D, DT, false, true)   \
        else CALL2(D, DT, false, false)              \
    }
    if (s.d == 64 && s.dtype == SPARGE_F16) CALL(64, SPARGE_F16)
    else if (s.d == 64 && s.dtype == SPARGE_BF16) CALL(64, SPARGE_BF16)
    else if (s.d == 128 && s.dtype == SPARGE_F16) CALL(128, SPARGE_F16)
    else if (s.d == 128 && s.dtype == SPARGE_BF16) CALL(128, SPARGE_BF16)
    else return hipErrorInvalidValue;
#undef CALL
#undef CALL2
#undef CALL3
    return hipGetLastError();
}

}  // namespace sparge
