// Stage (iii) with two waves per 32 queries, for launches with few workgroups.
#pragma once
#include "fp_attn.hpp"

namespace fp {

/*
 * The kernel of fp_attn.hpp gives a wave 32 queries, all keys of a tile and all dims of the output.  Here a pair of waves
 * shares that work: of a 64-key tile, wave p of the pair computes S^T and the probabilities of keys 32p..32p+31, the pair
 * exchanges probabilities (bf16, as the PV product takes them), row sums and row maxima through LDS, and wave p
 * accumulates half p of the output dims over all 64 keys.  No product is computed twice.  A workgroup has two pairs, 64
 * queries: twice the workgroups and twice the waves per query, with half the instructions in each wave's step.
 *
 * It is for launches that leave half the CUs idle, where the time is the longest row's chain of steps, and a step what one
 * wave per SIMD can issue: about 1700 cycles there (1024 of them matrix work), 1350 here.  Attention alone, both in turn on one
 * card, us: 4K tokens of 4 heads 28.3 -> 26.7 (whole pass 40.3 -> 38.1), 3000 tokens 23.3 -> 21.7, a 512-token chunk of 32 heads
 * behind 64K tokens 71.6 -> 67.6; rows of one or two blocks 0 to 1 us less.
 * The line is one workgroup per CU, 128 q-blocks.  Beyond it some CUs take two, and a launch whose rows are all long takes as long as
 * those: 160 q-blocks of 32 heads behind 32K tokens, 20 % of the blocks kept, 115.1 -> 160.5 (128: 113.9 -> 107.7; full attention 387 ->
 * 657, 128: 373 -> 370), at head dimension 64, where a CU holds two workgroups, 82.9 -> 90.4 (128: 83.3 -> 69.8).  Launches whose short
 * rows leave room for the second workgroup would gain beyond it (prompts of 160 q-blocks, 4 heads 40.6 -> 37.0, 32 heads 13.7 -> 12.6;
 * 192: 45.6 -> 41.4 and 15.2 -> 16.5), which the number of q-blocks alone does not tell.  At head dimension 256, where the LDS is
 * busiest, a form with two barriers a step was slower (517 -> 537).
 *
 * Every sum is formed from the same terms in the same order as there, and the reference point of the softmax moves on the same
 * tiles, so both kernels give the same bits: which of them runs may depend on the launch.
 *
 * One barrier per step: step t computes S^T of tile t+1, the exponentials of tile t and PV of tile t-1, whose probabilities
 * were published by the barrier of step t-1.  Exchange buffers are double (parity of the tile they belong to).
 */
constexpr int kPairs = 2;                          // pairs of waves per workgroup, 32 queries each
constexpr int kPairWaves = 2 * kPairs;
constexpr int kPairX = 4 * 1024;                   // probabilities of a pair: [16-key slice][lane] 16 B
constexpr int kPairL = 2 * 64 * 4;                 // row sums, or row maxima, of a pair: [wave][lane]
constexpr int kPairExchange = kPairX + 2 * kPairL; // of a pair and one parity
template <int D> constexpr int kPairXBase = (kAttnKBufs + kAttnVBufs) * kAttnTile<D, 64>;
template <int D> constexpr int kPairLds = kPairXBase<D> + 2 * kPairs * kPairExchange;   // 84 KB at D = 128

// V^T fragment v of this wave's half of the dims (16 keys v / (D/64), 32 dims v % (D/64) of the half).
template <int D>
__device__ __forceinline__ bf16x8 pair_vfrag(const char *smem, const uint32_t (&vaddr)[D / 64], int v) {
    const char *vp = smem + vaddr[v % (D / 64)] + 16 * (v / (D / 64)) * kAttnRowBytes<D>;
    const s16x4 lo = lds_read_tr(vp);
    const s16x4 hi = lds_read_tr(vp + 8 * kAttnRowBytes<D>);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// This lane's places in the exchange buffers, for one parity: its wave's slices, everybody's, its row sum and row max.
struct PairBufs {
    char *base;   // the pair's buffer of parity 0, + 16 l
    int p, l;
    __device__ __forceinline__ char *at(int par) const { return base + par * (kPairs * kPairExchange); }
    __device__ __forceinline__ void put_p(int par, int s, bf16x8 v) const { *reinterpret_cast<bf16x8 *>(at(par) + 2048 * p + 1024 * s) = v; }
    __device__ __forceinline__ bf16x8 get_p(int par, int s) const { return *reinterpret_cast<const bf16x8 *>(at(par) + 1024 * s); }
    __device__ __forceinline__ float *sums(int par) const { return reinterpret_cast<float *>(at(par) + kPairX - 16 * l) + l; }
    __device__ __forceinline__ void put_sum(int par, float v) const { sums(par)[64 * p] = v; }
    __device__ __forceinline__ float get_sum(int par) const { return sums(par)[0] + sums(par)[64]; }
    __device__ __forceinline__ void put_max(int par, float v) const { sums(par)[128 + 64 * p] = v; }
    __device__ __forceinline__ float other_max(int par) const { return sums(par)[128 + 64 * (1 - p)]; }
};

/*
 * One step, in slots as attn_step's: NKF that multiply a K fragment of tile t+1 (this wave's 32 keys), then NVF that
 * multiply a V^T fragment of tile t-1 (its half of the dims).  tm / tmo are the maxima of tile t over this wave's and the
 * other wave's keys; the first MFMA covers their last read.  The reference point for tile t moves before its exponentials, the
 * accumulator and the row sum, which then still lack tile t-1, behind PV of t-1.
 * X is the parity of tile t: its probabilities, sums and the maxima of tile t+1 go to buffers X, those of tile t-1 are in 1 - X.
 */
template <int D, int MODE, int X, int NL, class Load, class Sync, class Mask>
__device__ __forceinline__ void pair_step(const char *smem, uint32_t k1, uint32_t k2, const uint32_t (&va)[D / 64], const PairBufs &xb,
                                          const bf16x8 (&qb)[D / 16], f32x16 (&sc)[1], f32x16 (&sn)[1], f32x16 (&acc)[D / 64],
                                          float &m_run, float &l_run, float &tm, float &tmo, bf16x8 (&ring)[kAttnRing], float c,
                                          Load load, Sync sync, Mask mask) {
    constexpr int NDH = D / 64, NKF = D / 16, NVF = 4 * NDH, N = NKF + NVF, R = kAttnRing;
    constexpr int NES = N - R - 1;                                  // slots with exponentials: 1 .. NES
    constexpr int M0 = NKF + 1 < N - R ? NKF + 1 : N - R, NMS = N - R + 1 - M0;   // slots with the max: M0 .. N - R
    static_assert(N % R == 0 && NES >= 1, "the fragment ring comes round once per step");
    bf16x8 pb[2], pa[4];
    float x[16], ls[1], mc = 0.f, a = 1.f;
    bool moved = false;
    static_for<N>([&](auto f_) __attribute__((always_inline)) {
        constexpr int f = f_, nx = f + R - 1;
        if constexpr (nx == N) {
            sync();
            tmo = xb.other_max(X);
        }
        if constexpr (f == 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sn[0][i] = 0.f;
        }
        if constexpr (f < NKF) sn[0] = mfma32(ring[f % R], qb[f < NKF ? f : 0], sn[0]);
        else acc[(f - NKF) % NDH] = mfma32(ring[f % R], pa[(f - NKF) / NDH], acc[(f - NKF) % NDH]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (nx < NKF) ring[nx % R] = attn_kfrag<D, 32>(smem, k1, nx);
        else if constexpr (nx < N) ring[nx % R] = pair_vfrag<D>(smem, va, nx - NKF);
        else if constexpr (MODE != PEN) ring[nx % R] = attn_kfrag<D, 32>(smem, k2, nx - N);
        if constexpr (f >= 1 && f < 5 && f < NKF) pa[f - 1] = xb.get_p(1 - X, f - 1);
        if constexpr (f == NKF - 1) {
#pragma unroll
            for (int s = NKF - 2; s < 4; ++s) pa[s] = xb.get_p(1 - X, s);
        }
        if constexpr (f < NKF) static_for<NL * (f + 1) / NKF - NL * f / NKF>([&](auto i_) __attribute__((always_inline)) { load(NL * f / NKF + i_); });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (f == 0) {
            const float t = fmaxf(tm, tmo);
            moved = __ballot((t - m_run) * c > kAttnLazy);
            if (moved) {
                const float m_new = fmaxf(m_run, halves_max(t));
                a = fast_exp2((m_run - m_new) * c);
                m_run = m_new;
            }
            mc = m_run * c;
        }
        if constexpr (f >= 1 && f <= NES + 1) {
            constexpr int e0 = 16 * (f - 1) / NES, e1 = f <= NES ? 16 * f / NES : 16, d0 = f > 1 ? 16 * (f - 2) / NES : 0;
            attn_exp<32, e0, e1>(sc, c, mc, x);
            attn_exp_done<32, d0, e0>(x, ls, pb);
            if constexpr (d0 < 8 && e0 >= 8) xb.put_p(X, 0, pb[0]);
            if constexpr (d0 < 16 && e0 >= 16) {
                xb.put_p(X, 1, pb[1]);
                xb.put_sum(X, ls[0]);
            }
        }
        if constexpr (f == M0 && MODE != MAIN) mask();
        if constexpr (f == M0) tm = -INFINITY;
        if constexpr (f >= M0 && f < M0 + NMS) {
#pragma unroll
            for (int i = 8 * (f - M0) / NMS; i < 8 * (f - M0 + 1) / NMS; ++i) tm = max3(tm, sn[0][2 * i], sn[0][2 * i + 1]);
        }
        if constexpr (f == N - R) xb.put_max(X, tm);
        if constexpr (f == NKF) l_run += xb.get_sum(1 - X);
        __builtin_amdgcn_sched_barrier(0);
    });
    if (moved) {
        l_run *= a;
#pragma unroll
        for (int dt = 0; dt < NDH; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[dt][i] *= a;
    }
}

template <int D, bool SPARSE>
__global__ __launch_bounds__(64 * kPairWaves, 2) void attn_pair_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ cnt, const RowRec *__restrict__ rows_ranked,
    const int32_t *__restrict__ order, int item_order, int m_total, int n_max, int hq, int hkv, int g, int T, float c,
    uint16_t *__restrict__ O, float *__restrict__ lse) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int BLK = 128, KT = 64, TPB = BLK / KT;
    constexpr int NW = kPairWaves, QPG = 32 * kPairs, QS = BLK / QPG;   // waves, queries per workgroup, workgroups per q-block
    constexpr int KS = D / 16, NDH = D / 64;
    constexpr int RPL = kRowsPerLoad<D>, LPR = kChunks<D>, RB = kAttnRowBytes<D>;
    constexpr int RPW = KT / NW, LPT = RPW / RPL;          // tile rows per wave, wave-wide loads per wave and tile

    // work order, list and record as in attn_kernel
    const int xcd = blockIdx.x & 7, k0 = blockIdx.x >> 3;
    const int sub = k0 % QS, k = k0 / QS;
    const int hg = k % g;
    int hk, rank;
    if (!attn_item<false>(item_order, xcd, k / g, m_total, hkv, hk, rank)) return;
    hk = __builtin_amdgcn_readfirstlane(hk);       // held in scalar registers
    rank = __builtin_amdgcn_readfirstlane(rank);
    const int r = order[rank];
    const RowRec bi = rows_ranked[rank];
    const int h = hk * g + hg;
    const int I = bi.I;
    const int seq_tok0 = bi.k_tok0;
    const int last_tok = bi.k_end - 1;

    const int tid = threadIdx.x, l = tid & 63, half = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = w & 1, qw = w >> 1;                      // wave of the pair, pair
    const int q_local = 32 * qw + (l & 31);
    const int qoff = QPG * sub;
    const int q_len = bi.q_len - qoff < QPG ? bi.q_len - qoff : QPG;
    if (q_len <= 0) return;
    const int q_tok0 = bi.q_tok0 + qoff;

    int nb = I + 1, b0 = 0, b1 = 1;
    const int32_t *list = nullptr;
    if (SPARSE) {
        list = idx + ((size_t)h * m_total + r) * n_max;
        nb = cnt[(size_t)h * m_total + r];
        b0 = list[0];
        b1 = list[n_max > 1 ? 1 : 0];
        nb = nb < 0 ? 0 : (nb > I + 1 ? I + 1 : nb);
    }
    b0 = b0 < 0 ? 0 : (b0 > I ? I : b0);
    b1 = b1 < 0 ? 0 : (b1 > I ? I : b1);
    const int ntiles = TPB * nb;
    if (ntiles == 0) {   // empty list: O = 0, lse = -inf (uniform exit, before any barrier); wave p writes half p of the dims
        if (q_local < q_len) {
            uint16_t *op = O + ((size_t)(q_tok0 + q_local) * hq + h) * D + (D / 2) * p + (D / 4) * half;
            const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < D / 32; ++i) *reinterpret_cast<u32x4 *>(op + 8 * i) = z;
            if (lse != nullptr && half == 0 && p == 0) lse[(size_t)h * T + q_tok0 + q_local] = -INFINITY;
        }
        return;
    }
    const auto tile_block = [&](int t) __attribute__((always_inline)) { return attn_tile_block<SPARSE, TPB>(list, t, I, nb); };

    // Q^T B-fragments, as in attn_kernel (assembly: the prologue waits for them and the first K tile by count)
    bf16x8 qb[KS];
    {
        int row = q_local < q_len ? q_local : q_len - 1;
        const uint16_t *qp = Q + ((size_t)(q_tok0 + row) * hq + h) * D + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=&v"(qb[ks]) : "v"(qp), "n"(32 * ks) : "memory");
    }

    // Tile loads: wave w loads rows RPW w .. RPW w + RPW - 1 of a tile; otherwise as in attn_kernel.
    const uint32_t row_bytes = (uint32_t)hkv * D * 2;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(FP_LDS(char) *)smem;
    const uint32_t ld_dst = __builtin_amdgcn_readfirstlane(lds_base + RPW * w * RB);
    const int ld_row = RPW * w + l / LPR;   // + RPL i
    const int ld_pos = l % LPR;
    const char *Kb = reinterpret_cast<const char *>(K) + (size_t)hk * D * 2;
    const char *Vb = reinterpret_cast<const char *>(V) + (size_t)hk * D * 2;
    uint32_t ld_kcol[LPT], ld_vcol[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int row = ld_row + RPL * i;
        ld_kcol[i] = (uint32_t)((ld_pos ^ swz<D>(row)) * 16) + (uint32_t)row * row_bytes;
        ld_vcol[i] = (uint32_t)((ld_pos ^ (4 * attn_vswz<D>(row))) * 16) + (uint32_t)row * row_bytes;
    }
    // clamped load: every row is kept at or before the sequence's last token (keys past the end are masked as future)
    const auto load_tail = [&](const char *Xb, const uint32_t (&col)[LPT], int blk, int sub_tile, uint32_t ldsoff) __attribute__((always_inline)) {
        const int tok0 = seq_tok0 + blk * BLK + sub_tile * KT;
        const int base_tok = tok0 < last_tok ? tok0 : last_tok;
        const char *base = Xb + (size_t)base_tok * row_bytes;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(ld_dst + ldsoff);
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            int tok = tok0 + ld_row + RPL * i;
            tok = tok < last_tok ? tok : last_tok;
            load_to_lds(base, (uint32_t)(tok - base_tok) * row_bytes + (col[i] - (uint32_t)(ld_row + RPL * i) * row_bytes), dst + i * 1024);
        }
    };
#define FP_KBUF(par) ((uint32_t)((par) * kAttnTile<D, KT>))
#define FP_VBUF(par) ((uint32_t)(kAttnVBase<D, KT> + (par) * kAttnTile<D, KT>))
    const bool diag_full = seq_tok0 + (I + 1) * BLK - 1 <= last_tok;
    const int ent_max = diag_full ? I : I - 1;
#define FP_ENT_OFF(ent_, u)                                                                               \
    ((uint64_t)(uint32_t)(seq_tok0 + ((ent_) < 0 ? 0 : ((ent_) < ent_max ? (ent_) : ent_max)) * BLK + ((u) % TPB) * KT) * row_bytes)

    f32x16 acc[NDH];
#pragma unroll
    for (int dt = 0; dt < NDH; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float m_run, l_run = 0.f, tm = -INFINITY, tmo;

    // fragment addresses: attn_kernel's, K from this wave's 32 rows, V from its half of the dims
    const int krow = l & 31;
    const uint32_t k_frag = (uint32_t)((32 * p + krow) * RB + ((half ^ swz<D>(krow)) << 4));
    uint32_t v_frag[NDH];
    {
        const int e = (l & 15) >> 2, gq = (l & 31) >> 4, cc = l & 3;
        const uint32_t vb = (uint32_t)((4 * half + e) * RB + (2 * gq + (cc >> 1)) * 16 + 8 * (cc & 1));
#pragma unroll
        for (int i = 0; i < NDH; ++i) v_frag[i] = vb + (uint32_t)(((NDH * p + i) ^ attn_vswz<D>(e)) * 64);
    }
    const PairBufs xb = {smem + kPairXBase<D> + qw * kPairExchange + 16 * l, p, l};
    const auto lim_of = [&](int t) __attribute__((always_inline)) {   // causal limit for this lane's keys of tile t
        return tile_block(t) == I ? qoff + q_local - (t % TPB) * KT - 32 * p - 4 * half : 2 * KT;
    };

    // Prologue: this wave's half of S^T of tile 0 and the row max of both halves; then step 0, which has no PV.
    load_tail(Kb, ld_kcol, b0, 0, FP_KBUF(0));
    load_tail(Kb, ld_kcol, b0, 1, FP_KBUF(1));
    load_tail(Vb, ld_vcol, b0, 0, FP_VBUF(0));
    FP_WAIT_VMCNT(2 * LPT);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qb[ks]));
    __syncthreads();
    f32x16 sA[1], sB[1];
    bf16x8 ring[kAttnRing];
    const auto scores = [&](uint32_t kb, f32x16 (&s)[1]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[0][i] = 0.f;
        static_for<KS>([&](auto f_) __attribute__((always_inline)) { s[0] = mfma32(attn_kfrag<D, 32>(smem, kb + k_frag, f_), qb[f_], s[0]); });
    };
    const auto exps = [&](const f32x16 (&s)[1], int par) __attribute__((always_inline)) {
        bf16x8 pb[2];
        float x[16], ls[1];
        attn_exp<32, 0, 16>(s, c, m_run * c, x);
        attn_exp_done<32, 0, 16>(x, ls, pb);
        xb.put_p(par, 0, pb[0]);
        xb.put_p(par, 1, pb[1]);
        xb.put_sum(par, ls[0]);
    };
    const auto pv = [&](uint32_t vb, int par) __attribute__((always_inline)) {
        uint32_t va[NDH];
#pragma unroll
        for (int i = 0; i < NDH; ++i) va[i] = vb + v_frag[i];
        bf16x8 pa[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) pa[s] = xb.get_p(par, s);
        l_run += xb.get_sum(par);
#pragma unroll
        for (int v = 0; v < 4 * NDH; ++v) acc[v % NDH] = mfma32(pair_vfrag<D>(smem, va, v), pa[v / NDH], acc[v % NDH]);
    };
    scores(FP_KBUF(0), sA);
    attn_mask<32>(sA, b0 == I ? qoff + q_local - 32 * p - 4 * half : 2 * KT);
    tm = attn_rowmax_half<32>(sA);
    xb.put_max(1, tm);
    FP_WAIT_VMCNT(0);
    __syncthreads();
    tmo = xb.other_max(1);
    m_run = halves_max(fmaxf(tm, tmo));   // finite: key 0 of tile 0 is visible to every query
    if (ntiles > 2) load_tail(Kb, ld_kcol, tile_block(2), 2 % TPB, FP_KBUF(0));
    else load_tail(Vb, ld_vcol, b0, 1, FP_KBUF(0));   // see the last tile
    scores(FP_KBUF(1), sB);
    exps(sA, 0);
    attn_mask<32>(sB, lim_of(1));
    tm = attn_rowmax_half<32>(sB);
    xb.put_max(0, tm);
    FP_WAIT_VMCNT(0);
    __syncthreads();
    tmo = xb.other_max(0);
    if (ntiles > 2) {
#pragma unroll
        for (int f = 0; f < kAttnRing - 1; ++f) ring[f] = attn_kfrag<D, 32>(smem, FP_KBUF(0) + k_frag, f);
    }

    // Step t, from 1 on, loads K[t+2] into the buffer of K[t] and V[t] into that of V[t-2].  Variants as in attn_kernel; the last
    // step (PEN) loads no K but V of the last tile as well, into the K buffer that is free by then.  Steps come in pairs that start
    // at an odd t: S^T of tile t is in sB.
#define FP_STEP(MODE, PAR, t, sc, sn, LOADX)                                                               \
    do {                                                                                                  \
        const int t_ = (t);                                                                               \
        uint32_t va_[NDH];                                                                                \
        _Pragma("unroll") for (int i_ = 0; i_ < NDH; ++i_) va_[i_] = FP_VBUF(1 - (PAR)) + v_frag[i_];     \
        pair_step<D, MODE, PAR, 2 * LPT>(                                                                 \
            smem, FP_KBUF(1 - (PAR)) + k_frag, FP_KBUF(PAR) + k_frag, va_, xb, qb, sc, sn, acc, m_run, l_run, tm, tmo, ring, c, LOADX, \
            [&]() __attribute__((always_inline)) { FP_WAIT_VMCNT(0); __syncthreads(); },                  \
            [&]() __attribute__((always_inline)) { attn_mask<32>(sn, lim_of(t_ + 1)); });                 \
    } while (0)
    // load i of a step, K first; KOFF / VOFF are the byte offsets of tiles t+2 / t
#define FP_LOAD_MAIN(PAR, KOFF, VOFF)                                                                      \
    [&](int i_) __attribute__((always_inline)) {                                                          \
        const bool k_ = i_ < LPT;                                                                         \
        const int j_ = k_ ? i_ : i_ - LPT;                                                                \
        load_to_lds(k_ ? Kb + (KOFF) : Vb + (VOFF), k_ ? ld_kcol[j_] : ld_vcol[j_],                       \
                    ld_dst + (k_ ? FP_KBUF(PAR) : FP_VBUF(PAR)) + j_ * 1024);                             \
    }
#define FP_LOAD_TAIL(PAR, t, IS_PEN)                                                                       \
    [&](int i_) __attribute__((always_inline)) {                                                          \
        if (i_ == 0 && !(IS_PEN)) load_tail(Kb, ld_kcol, tile_block((t) + 2), ((t) + 2) % TPB, FP_KBUF(PAR)); \
        if (i_ == 0 && (IS_PEN)) load_tail(Vb, ld_vcol, tile_block((t) + 1), ((t) + 1) % TPB, FP_KBUF(PAR)); \
        if (i_ == LPT) load_tail(Vb, ld_vcol, tile_block(t), (t) % TPB, FP_VBUF(PAR));                    \
    }
    const int n_plain = tile_block(ntiles - 1) == I ? TPB * (nb - 1) : ntiles;
    int t = 1;
    if (t + 3 < n_plain) {
        // Tiles t+2 (odd: second of its block) and t+3 (first of the next one) of K, t and t+1 of V: three neighbouring blocks,
        // whose offsets are carried; the next list entry is fetched a pair of steps before it is needed.
        uint64_t oa = FP_ENT_OFF(b0, 0), ob = FP_ENT_OFF(b1, 0);
        int e = tile_block(4);
        const uint64_t second = (uint64_t)KT * row_bytes;
        for (; t + 3 < n_plain; t += 2) {
            const uint64_t oc = FP_ENT_OFF(e, 0);
            const int u = (t + 5) / TPB < nb ? (t + 5) / TPB : nb - 1;
            e = SPARSE ? list[u] : u;
            FP_STEP(MAIN, 1, t, sB, sA, FP_LOAD_MAIN(1, ob + second, oa + second));
            FP_STEP(MAIN, 0, t + 1, sA, sB, FP_LOAD_MAIN(0, oc, ob));
            oa = ob;
            ob = oc;
        }
    }
    for (; t < ntiles - 3; t += 2) {
        FP_STEP(TAIL, 1, t, sB, sA, FP_LOAD_TAIL(1, t, false));
        FP_STEP(TAIL, 0, t + 1, sA, sB, FP_LOAD_TAIL(0, t + 1, false));
    }
    if (ntiles > 2) {
        FP_STEP(TAIL, 1, t, sB, sA, FP_LOAD_TAIL(1, t, false));
        FP_STEP(PEN, 0, t + 1, sA, sB, FP_LOAD_TAIL(0, t + 1, true));
    }
    // The last two tiles' PV; the reference point for the last tile moves behind the first of them, as in a step.
    {
        const float tl = fmaxf(tm, tmo), m_old = m_run;
        const bool moved = __ballot((tl - m_run) * c > kAttnLazy);
        if (moved) m_run = fmaxf(m_run, halves_max(tl));
        exps(sB, 1);
        pv(FP_VBUF(0), 0);
        if (moved) {
            const float a = fast_exp2((m_old - m_run) * c);
            l_run *= a;
#pragma unroll
            for (int dt = 0; dt < NDH; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[dt][i] *= a;
        }
        __syncthreads();
        pv(FP_KBUF(0), 1);
        __syncthreads();   // the output goes through the K buffers
    }

    // O and lse.  The wave's 32 x D/2 output tile is turned through its own part of the K buffers (no reader and no load is
    // left there); chunk c of row q at chunk c ^ (q & mask).
    const float l_tot = halves_sum(l_run);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    {
        constexpr int HB = D, HC = D / 16, MASK = HC - 1;   // bytes and 16-byte chunks of half a row
        static_assert(HC <= 16 && NW * 32 * HB <= kAttnVBase<D, KT>, "fits the K buffers");
        char *ob = smem + w * (32 * HB);
        const int qrow = l & 31;
#pragma unroll
        for (int dt = 0; dt < NDH; ++dt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[dt][4 * q4 + e] * inv);
                *reinterpret_cast<bf16x4 *>(ob + qrow * HB + (((4 * dt + q4) ^ (qrow & MASK)) << 4) + 8 * half) = o;
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int pc = l % HC;
#pragma unroll
        for (int i = 0; i < 32 * HC / 64; ++i) {
            const int orow = (64 / HC) * i + l / HC;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(ob + orow * HB + (pc << 4));
            if (32 * qw + orow < q_len)
                *reinterpret_cast<u32x4 *>(O + ((size_t)(q_tok0 + 32 * qw + orow) * hq + h) * D + (D / 2) * p + ((pc ^ (orow & MASK)) << 3)) = v;
        }
    }
    if (q_local < q_len && lse != nullptr && half == 0 && p == 0)
        lse[(size_t)h * T + q_tok0 + q_local] = l_tot > 0.f ? m_run * c + __log2f(l_tot) : -INFINITY;
#undef FP_LOAD_MAIN
#undef FP_LOAD_TAIL
#undef FP_ENT_OFF
#undef FP_KBUF
#undef FP_VBUF
#undef FP_STEP
}

}  // namespace fp
