// Stage (iii): index-driven block-sparse attention (Sec. 3.5, Alg. 3) and, from the same
// template, full causal attention.  bf16 MFMA for both contractions, fp32 online softmax.
#pragma once
#include "fp_device.hpp"
#include "fp_order.hpp"

namespace fp {

// LDS: two K buffers and two V buffers of one 64-key tile (64 rows x 2D bytes, unpadded) each.
// Tiles are written by direct global->LDS loads (16 B per lane, lane i lands at base + 16 i), so
// bank conflicts are avoided by permuting the 16-byte chunks inside a row instead of padding
// (stated for head dimension 128, 16 chunks per row; at 64 a row is half a turn of the banks long, so that two neighbouring
// rows share a value and r/2 takes the place of r: with r itself rows eight apart met in K and two apart in V, and half of
// the LDS unit's active cycles were conflicts; 16K tokens 274.7 -> 273.9 us, the vector work bounds it):
//   K row r keeps chunk c at position c ^ (r & 15): the A-fragment reads of 16 consecutive rows
//     at one chunk index then hit 16 different bank groups;
//   V row r keeps chunk c at position c ^ 4 (r & 3): the four rows a transpose read touches per
//     lane group then hit four different 64-byte bank groups.
// Head dimension 128: 16 KB tiles, 64 KB, two workgroups per CU (registers).  64: 32 KB, three (full attention, 16K tokens:
// 1151 us with two, 1137 with three).
// 256: 32 KB tiles, 128 KB, one workgroup (its accumulators and query fragments need 512 registers).
// A workgroup has one wave per 32 queries of its q-block part, four at most; a 64-query block gets
// two waves and 32-key tiles (32 KB, four workgroups per CU), so that every wave still loads 16
// rows of each tile and no wave repeats another's queries.
template <int BLK> constexpr int kAttnWaves = BLK < 128 ? BLK / 32 : 4;
template <int BLK> constexpr int kAttnTileKeys = 16 * kAttnWaves<BLK>;
template <int D> constexpr int kAttnRowBytes = 2 * D;
template <int D, int KT> constexpr int kAttnTile = KT * kAttnRowBytes<D>;   // 16384 at D = 128, 64 keys
constexpr int kAttnKBufs = 2, kAttnVBufs = 2;
template <int D, int KT> constexpr int kAttnVBase = kAttnKBufs * kAttnTile<D, KT>;
template <int D, int BLK> constexpr int kAttnLds = (kAttnKBufs + kAttnVBufs) * kAttnTile<D, kAttnTileKeys<BLK>>;   // 65536 at D = 128
template <int D> __device__ __forceinline__ constexpr int attn_vswz(int r) { return D < 128 ? (r >> 1) & 1 : r & 3; }   // V rows: chunk ^ 4 attn_vswz(r)

// ds_read_b64_tr_b16: within each group of 16 lanes the 16 x 4 b16 values addressed by the
// lanes (lane j supplies 4 consecutive b16) are exchanged so that lane i receives, in element e,
// the value that lane 4e + i/4 addressed at position i%4.  With lane j pointing at row (j/4)
// and columns 4*(j%4)..+3 of a row-major 4 x 16 patch, lane i ends up with column i of the four
// rows: exactly the key-contiguous fragment the PV product needs from a row-major V tile.
__device__ __forceinline__ s16x4 lds_read_tr(const char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((FP_LDS(s16x4) *)(FP_LDS(char) *)p);
}

/*
 * One workgroup (4 waves) per (query head, q-block row); wave w owns queries 32w..32w+31 of the
 * block.  Alg. 3's loop over the listed blocks runs as a loop over 64-key tiles (two per block)
 * whose addresses come straight from the index list: an unlisted block costs no instruction.
 * (Other block sizes: a 256-query block is two such workgroups over four tiles per block, a
 * 64-query block one workgroup of two waves over two 32-key tiles per block; the counts below are
 * for 64-key tiles.)
 *
 * Per tile and wave:
 *   S^T = K Q^T  (keys x queries, 16 MFMA 32x32x16): the query index is the lane column, so the
 *         row max and row sum of the softmax are reductions over a lane's own registers plus one
 *         exchange between the wave's halves;
 *   causal mask only if the tile belongs to the diagonal block (Alg. 3, is_diag);
 *   online softmax in base 2: p = 2^(c*s - c*m) with m a reference point that follows the row
 *         max lazily (see attn_new_max), so the accumulator is rescaled a few times per row;
 *   O^T += V^T P^T (16 MFMA): P^T is already in B-operand layout (registers of S^T, packed to
 *         bf16), V^T fragments come from the row-major V tile through LDS transpose reads.
 *
 * Software pipeline inside the wave: step t issues the QK^T MFMAs of tile t+1 with the softmax of
 * tile t (VALU) between them, then the PV MFMAs of tile t with the max of tile t+1 between
 * them.  The S^T registers alternate between two sets (steps are unrolled in pairs).  K runs one tile
 * ahead of V in LDS: step t reads K[t+1] and V[t] and issues the direct-to-LDS loads of K[t+2] and
 * V[t+1]; two buffers each, one barrier per step.  The order inside a step is fixed in the source (attn_step).
 *
 * Work order: blockIdx -> (XCD, slot), see attn_item.  The g query heads of a super-item (KV head, row) are neighbouring slots of
 * one XCD: they run at about the same time and find each other's K/V tiles in its L2.
 */
// Block of key tile t: entry t / TPB of the list (TPB tiles per block), the entry index kept
// below nb and the block id inside [0, I].
template <bool SPARSE, int TPB>
__device__ __forceinline__ int attn_tile_block(const int32_t *list, int t, int I, int nb) {
    int li = t / TPB;
    li = li < nb ? li : nb - 1;
    if (!SPARSE) return li;
    const int b = list[li];
    return b < 0 ? 0 : (b > I ? I : b);
}

// Head dimension 256 runs one wave per SIMD on all 512 registers: the accumulators and the query fragments
// belong in the accumulation half of the file, S^T and everything the vector ALU touches in the other.
// The compiler gives every MFMA result of such a kernel an accumulation register, so the S^T MFMAs are written out.
template <int D> constexpr bool kAttnAgpr = D > 128;

// Whether a lane's load offsets include the row of each load (one vector instruction less per load).  At head dimension 256,
// with twice the loads per tile, the addition stays in the wait state of the load (16K tokens 2 % slower without it).
template <int D> constexpr bool kAttnRowInOffset = D <= 128;

// One MFMA of S^T = K Q^T; FIRST starts from zero.  An operand that a vector instruction wrote (a register copy: the
// fragments come from loads) needs two wait states before the MFMA, which the compiler does not give to assembly.
#define FP_MFMA(C) "v_mfma_f32_32x32x16_bf16 %[d], %[a], %[q], " C
template <int D, bool FIRST>
__device__ __forceinline__ void attn_mfma_s(f32x16 &s, bf16x8 a, bf16x8 q) {
    if constexpr (kAttnAgpr<D>) {
        if constexpr (FIRST) asm volatile("s_nop 1\n\t" FP_MFMA("0") : [d] "=&v"(s) : [a] "v"(a), [q] "a"(q));
        else asm volatile("s_nop 1\n\t" FP_MFMA("%[d]") : [d] "+v"(s) : [a] "v"(a), [q] "a"(q));
    } else {
        if (FIRST) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = 0.f;
        }
        s = mfma32(a, q, s);
    }
}

// Wait states between the last of these MFMAs and the first vector instruction that touches the result, where no
// other MFMAs lie between (the compiler takes care of its own MFMAs, not of assembly).
template <int D, int KT>
__device__ __forceinline__ void attn_settle(f32x16 (&s)[KT / 32]) {
    if constexpr (kAttnAgpr<D>) {
#pragma unroll
        for (int kt = 0; kt < KT / 32; ++kt) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s[kt]));
    }
}

// The same where N MFMAs of the compiler's lie between: only the reads of the result are held behind this point.
template <int D, int KT, int N>
__device__ __forceinline__ void attn_settled_by_pv(f32x16 (&s)[KT / 32]) {
    if constexpr (kAttnAgpr<D>) {
        static_assert(N >= 3, "8 wait states each, one after another: the third starts past the 20 a result needs at most");
#pragma unroll
        for (int kt = 0; kt < KT / 32; ++kt) asm volatile("" : "+v"(s[kt]));
    }
}

// K fragment f of a tile (k-slice f / (KT/32), 32 keys f % (KT/32)).
template <int D, int KT>
__device__ __forceinline__ bf16x8 attn_kfrag(const char *smem, uint32_t kaddr, int f) {
    constexpr int NKT = KT / 32;
    return *reinterpret_cast<const bf16x8 *>(smem + (kaddr ^ (uint32_t)((f / NKT) << 5)) + 32 * (f % NKT) * kAttnRowBytes<D>);
}
// V^T fragment v of a tile (16 keys v / (D/32), 32 dims v % (D/32)).
template <int D>
__device__ __forceinline__ bf16x8 attn_vfrag(const char *smem, const uint32_t (&vaddr)[D / 32], int v) {
    const char *vp = smem + vaddr[v % (D / 32)] + 16 * (v / (D / 32)) * kAttnRowBytes<D>;
    const s16x4 lo = lds_read_tr(vp);
    const s16x4 hi = lds_read_tr(vp + 8 * kAttnRowBytes<D>);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Causal mask of a diagonal tile: key 32 kt + 8(i/4) + i%4 (element i of s[kt]) is in this lane's future if it
// exceeds lim = query - tile offset - 4*half.
template <int KT>
__device__ __forceinline__ void attn_mask(f32x16 (&s)[KT / 32], int lim) {
#pragma unroll
    for (int kt = 0; kt < KT / 32; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (32 * kt + 8 * (i >> 2) + (i & 3) > lim) s[kt][i] = -INFINITY;
}

// Row max over this lane's half of one tile's S^T.
template <int KT>
__device__ __forceinline__ float attn_rowmax_half(const f32x16 (&s)[KT / 32]) {
    float t = fmaxf(s[0][0], s[0][1]);
#pragma unroll
    for (int i = 2; i < KT / 2; i += 2) t = max3(t, s[i >> 4][i & 15], s[i >> 4][(i & 15) + 1]);
    return t;
}

// Online-softmax bookkeeping for a new tile.  tm is the largest logit among this lane's own keys of the tile: lanes
// l and l ^ 32 hold the two halves of a row.  m_run is the reference point of the
// exponentials, not necessarily the true running max: it is moved (and the accumulator and the
// row sum rescaled) only when some row's max has outgrown it by more than kAttnLazy in the base-2
// exponent (wave-uniform test).  Until then p = 2^(c*s - c*m_run) may reach 2^kAttnLazy, which
// fp32 sums and bf16 operands hold without loss; O = acc / l and lse = c*m_run + log2 l do not
// depend on the reference point.  With 32 rows per wave an exact-max rule would fire on most
// tiles of a short row; this one fires a few times per row at most.
// A row's max outgrows the reference where one of its halves does, so the test takes the halves as they are and the
// exchange between them, a serial chain at the end of every step, is left to the rare branch (same decisions; 4K tokens
// of 4 heads 30.1 -> 29.5 us, 8K 198.9 -> 196.3, 128K 6993 -> 6926, block 64 at 32K 1022 -> 1011).
constexpr float kAttnLazy = 8.0f;
template <int NDT>
__device__ __forceinline__ void attn_new_max(float tm, float c, float &m_run, float &l_run, f32x16 (&acc)[NDT]) {
    if (__ballot((tm - m_run) * c > kAttnLazy)) {
        const float m_new = fmaxf(m_run, halves_max(tm));
        const float a = fast_exp2((m_run - m_new) * c);
        l_run *= a;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[dt][i] *= a;
        m_run = m_new;
    }
}

// Exponentials E0 .. E1-1 of a tile in the order in which the PV product needs them (element e: 16-key slice
// e / 8): x = 2^(c*s - c*m).  They are finished by attn_exp_done, one slot of the step later, so that
// nothing waits for the transcendental unit.  Written as assembly so that each stays in its slot.  The compiler
// does not see what is inside:
//   - the result of v_exp_f32 needs one wait state before a vector instruction reads it: the next element's
//     v_fma_f32 (after the last one a wait) stands behind it in the same statement;
//   - the MFMA results in s need none here: they come behind a branch on the row max of the whole tile (attn_new_max), so
//     that instructions the compiler does see (at head dimension 256: attn_settle, or the PV MFMAs before
//     the max) have waited for every element before.
#define FP_FMA(x, s) "v_fma_f32 %[" x "], %[" s "], %[c], -%[mc]\n\t"
#define FP_EXP "v_exp_f32 %[x], %[x]\n\t"
template <int KT, int E0, int E1>
__device__ __forceinline__ void attn_exp(const f32x16 (&s)[KT / 32], float c, float mc, float (&x)[KT / 2]) {
    static_for<E1 - E0>([&](auto i_) __attribute__((always_inline)) {
        constexpr int e = E0 + i_, n = e + 1 < KT / 2 ? e + 1 : e;
        const float se = s[e >> 4][e & 15], sn = s[n >> 4][n & 15];
        float &xe = x[e], &xn = x[n];
        if constexpr (e == 0) asm volatile(FP_FMA("x", "s") FP_EXP FP_FMA("y", "t") : [x] "=&v"(xe), [y] "=&v"(xn) : [s] "v"(se), [t] "v"(sn), [c] "s"(c), [mc] "v"(mc));
        else if constexpr (n > e) asm volatile(FP_EXP FP_FMA("y", "t") : [x] "+v"(xe), [y] "=&v"(xn) : [t] "v"(sn), [c] "s"(c), [mc] "v"(mc));
        else asm volatile(FP_EXP "s_nop 0" : [x] "+v"(xe));
    });
}
// Exponential E and one MFMA of S^T in one statement, for head dimension 256: the vector instructions are the MFMA's
// wait states.
template <int KT, bool FIRST, int E>
__device__ __forceinline__ void attn_exp_mfma(f32x16 &d, bf16x8 a, bf16x8 q, const f32x16 (&s)[KT / 32], float c, float mc,
                                              float (&x)[KT / 2]) {
    static_assert(E + 1 < KT / 2 && (!FIRST || E == 0), "a tile starts with the first MFMAs of its S^T and ends beside the PV MFMAs");
    const float se = s[E >> 4][E & 15], sn = s[(E + 1) >> 4][(E + 1) & 15];
    float &xe = x[E], &xn = x[E + 1];
    if constexpr (FIRST)
        asm volatile(FP_FMA("x", "s") FP_EXP FP_FMA("y", "t") FP_MFMA("0")
                     : [x] "=&v"(xe), [y] "=&v"(xn), [d] "=&v"(d) : [s] "v"(se), [t] "v"(sn), [c] "s"(c), [mc] "v"(mc), [a] "v"(a), [q] "a"(q));
    else if constexpr (E == 0)
        asm volatile(FP_FMA("x", "s") FP_EXP FP_FMA("y", "t") FP_MFMA("%[d]")
                     : [x] "=&v"(xe), [y] "=&v"(xn), [d] "+v"(d) : [s] "v"(se), [t] "v"(sn), [c] "s"(c), [mc] "v"(mc), [a] "v"(a), [q] "a"(q));
    else
        asm volatile(FP_EXP FP_FMA("y", "t") FP_MFMA("%[d]")
                     : [x] "+v"(xe), [y] "=&v"(xn), [d] "+v"(d) : [t] "v"(sn), [c] "s"(c), [mc] "v"(mc), [a] "v"(a), [q] "a"(q));
}
#undef FP_FMA
#undef FP_EXP
#undef FP_MFMA
// Row sum, over the fp32 values before rounding so that lse does not inherit bf16's 2^-9, and
// rounding to the B operand of the PV product.  One chain of additions per 32 keys, started afresh in every
// tile: a chain that went on from the running sum would round it once per key instead of once per tile.
template <int KT, int E0, int E1>
__device__ __forceinline__ void attn_exp_done(const float (&x)[KT / 2], float (&ls)[KT / 32], bf16x8 (&pb)[KT / 16]) {
#pragma unroll
    for (int e = E0; e < E1; ++e) {
        ls[e >> 4] = (e & 15) ? ls[e >> 4] + x[e] : x[e];
        pb[e >> 3][e & 7] = (__bf16)x[e];
    }
}
template <int KT>
__device__ __forceinline__ float attn_tile_sum(const float (&ls)[KT / 32]) {
    if constexpr (KT > 32) return ls[0] + ls[1];
    else return ls[0];
}

/*
 * One step: QK^T of tile t+1 (into sn), softmax and PV of tile t (from sc).  On entry the row max of
 * tile t is folded into m_run, K[t+1] and V[t] are complete in LDS and `ring` holds the first
 * kAttnRing - 1 fragments of K[t+1].
 *
 * The step is a fixed sequence of slots, one per fragment: NKF slots that multiply a K fragment, then NVF that
 * multiply a V^T fragment.  A slot issues its MFMA, reads the fragment needed kAttnRing - 1 slots later
 * and does a share of the vector work (in this order: behind an MFMA a wave's next vector instruction waits for some
 * 16 cycles, which the reads and the tile loads do not): exponentials of tile t beside the QK^T MFMAs (those of the last 16 keys
 * beside the first PV MFMAs, which do not need them yet), the max of tile t+1 beside the later PV MFMAs.
 * Scheduling fences keep the slots apart.  Left to itself the compiler asks for a fragment right
 * before its MFMA and waits there, and bunches the vector work: a wave then stalls on LDS at
 * every MFMA, which the other wave of the SIMD hides in part at head dimension 128 and no wave hides at 256.
 *
 * `load(i)`, i < NL, issues the tile loads, spread evenly over the QK^T slots (two per slot from the start of the step filled
 * the address unit's queue and the wave waited for it: head dimension 256, dense 8K 492 -> 480 us; 128: 8K sparse 188.9 -> 184.3); they go into the
 * buffers of K[t] and V[t-1], whose last readers are behind the barrier of step t-1.  That barrier
 * (`sync`: wait for the loads, workgroup barrier) sits where the last V fragment of the step has been read
 * and kAttnRing - 1 PV slots are still to come, which cover the first reads of the next K tile.
 *
 * Measured against the compiler's own order with three K buffers (attention alone, launches back to back, both in turn
 * on one card, us): head dimension 256, 16K tokens 654 -> 561, dense 8K 633 -> 547; 128: 4K tokens of 4 heads 35.3 -> 30.4,
 * 32K tokens 1425 -> 1357, dense 32K 7992 -> 7801; 64: 16K tokens 275 -> 268; block 64: 32K tokens 1047 -> 997; block 256:
 * 1994 -> 1897.  Long rows at head dimension 128 gain least because the clock sets most of their rate: on all-zero inputs
 * the same launch of dense 32K takes 1 / 1.71 of the time (64: 1 / 1.51, 256: 1 / 1.45, 16K tokens).
 */
constexpr int kAttnRing = 4;
enum { MAIN = 0, TAIL = 1, PEN = 2 };   // see the kernel
template <int D, int KT, int MODE, class Load, class Sync, class Mask>
__device__ __forceinline__ void attn_step(const char *smem, uint32_t k1, uint32_t k2, const uint32_t (&va)[D / 32],
                                          const bf16x8 (&qb)[D / 16], const f32x16 (&sc)[KT / 32], f32x16 (&sn)[KT / 32],
                                          f32x16 (&acc)[D / 32], float &m_run, float &l_run, bf16x8 (&ring)[kAttnRing], float c,
                                          Load load, Sync sync, Mask mask) {
    constexpr int NDT = D / 32, NKT = KT / 32, NKF = NKT * D / 16, NVF = KT / 16 * NDT, R = kAttnRing, NL = 2 * NDT;
    constexpr int NE = KT / 2, EQK = NE - 8, NQS = NKF - 1;   // exponentials of the tile; those beside the QK^T MFMAs and their slots
    constexpr int MS = KT > 32 ? NVF / 2 : NVF / 2 - 1;   // PV slots with exponentials; the max follows
    constexpr int MU = NVF - MS - (R - 1), NM = KT / 4;   // slots of the max, operations in it
    static_assert((NKF + NVF) % R == 0, "the fragment ring comes round once per step");
    static_assert(MS < NVF - NDT, "the last 16 keys' probabilities are complete before their first PV slot");
    bf16x8 pb[KT / 16];
    float x[NE], ls[NKT], tm = -INFINITY;
    const float mc = m_run * c;
    static_for<NKF>([&](auto f_) __attribute__((always_inline)) {
        constexpr int f = f_, nx = f + R - 1, e0 = EQK * f / NQS, e1 = f < NQS ? EQK * (f + 1) / NQS : EQK;
        if constexpr (kAttnAgpr<D> && e1 > e0) attn_exp_mfma<KT, (f < NKT), e0>(sn[f % NKT], ring[f % R], qb[f / NKT], sc, c, mc, x);
        else attn_mfma_s<D, (f < NKT)>(sn[f % NKT], ring[f % R], qb[f / NKT]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (nx < NKF) ring[nx % R] = attn_kfrag<D, KT>(smem, k1, nx);
        else ring[nx % R] = attn_vfrag<D>(smem, va, nx - NKF);
        static_for<NL * (f + 1) / NKF - NL * f / NKF>([&](auto i_) __attribute__((always_inline)) { load(NL * f / NKF + i_); });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kAttnAgpr<D>) attn_exp<KT, e0, e1>(sc, c, mc, x);
        else static_assert(e1 - e0 <= 1, "attn_exp_mfma takes one exponential");
        if constexpr (f > 0) attn_exp_done<KT, EQK * (f - 1) / NQS, e0>(x, ls, pb);
        __builtin_amdgcn_sched_barrier(0);
    });
    static_for<NVF>([&](auto v_) __attribute__((always_inline)) {
        constexpr int v = v_, nx = v + R - 1;
        if constexpr (nx == NVF) sync();
        acc[v % NDT] = mfma32(ring[(NKF + v) % R], pb[v / NDT], acc[v % NDT]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (nx < NVF) ring[(NKF + nx) % R] = attn_vfrag<D>(smem, va, nx);
        else if constexpr (MODE != PEN) ring[(NKF + nx) % R] = attn_kfrag<D, KT>(smem, k2, nx - NVF);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (v <= MS) {
            constexpr int e0 = EQK + 8 * v / MS, e1 = v < MS ? EQK + 8 * (v + 1) / MS : NE;
            attn_exp<KT, e0, e1>(sc, c, mc, x);
            attn_exp_done<KT, (v == 0 ? EQK : EQK + 8 * (v - 1) / MS), e0>(x, ls, pb);
        }
        if constexpr (v == MS + 1) l_run += attn_tile_sum<KT>(ls);
        if constexpr (MODE == MAIN && v == MS) attn_settled_by_pv<D, KT, MS>(sn);
        if constexpr (MODE == MAIN && v >= MS) {
#pragma unroll
            for (int i = NM * (v - MS) / MU; i < (v - MS < MU ? NM * (v - MS + 1) / MU : NM); ++i)
                tm = max3(tm, sn[(2 * i) >> 4][(2 * i) & 15], sn[(2 * i + 1) >> 4][(2 * i + 1) & 15]);
        }
        if constexpr (MODE != MAIN && v == MS) {
            mask();
            tm = attn_rowmax_half<KT>(sn);
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    attn_new_max<NDT>(tm, c, m_run, l_run, acc);
}

template <int D, int BLK, bool SPARSE>
__global__ __launch_bounds__(64 * kAttnWaves<BLK>, D > 128 ? 1 : D < 128 ? 3 : 2) void attn_kernel(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ cnt, const RowRec *__restrict__ rows_ranked,
    const int32_t *__restrict__ order, int item_order, int m_total, int n_max, int hq, int hkv, int g, int T, float c,
    uint16_t *__restrict__ O, float *__restrict__ lse) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int KS = D / 16;            // k-slices of the QK^T contraction
    constexpr int NDT = D / 32;           // 32-wide tiles of the head dimension in the output
    constexpr int KT = kAttnTileKeys<BLK>;   // keys per tile: 64, or 32 for the two-wave workgroup of a 64-query block
    constexpr int LPT = D / 32;           // wave-wide 1 KB loads per wave and tile (16 rows per wave)
    constexpr int RPL = kRowsPerLoad<D>;  // rows one such load covers
    constexpr int LPR = kChunks<D>;       // lanes (= 16-byte chunks) per row
    constexpr int RB = kAttnRowBytes<D>;
    constexpr int TPB = BLK / KT;                     // key tiles per key block: 2 or 4
    constexpr int QS = BLK > 128 ? BLK / 128 : 1;     // workgroups per (head, q-block), 128 queries each
    static_assert(TPB % 2 == 0, "the two register sets of the pipeline alternate over an even tile count");

    const int x = blockIdx.x & 7, k0 = blockIdx.x >> 3;
    const int sub = k0 % QS, k = k0 / QS;             // which 128 queries of the q-block
    const int hg = k % g;
    int hk, rank;
    if (!attn_item<SPARSE>(item_order, x, k / g, m_total, hkv, hk, rank)) return;
    hk = __builtin_amdgcn_readfirstlane(hk);       // held in scalar registers
    rank = __builtin_amdgcn_readfirstlane(rank);
    const int r = order[rank];               // both tables are indexed by rank: one round trip
    const RowRec bi = rows_ranked[rank];
    const int h = hk * g + hg;
    const int I = bi.I;                  // diagonal key block (q-block index + KV prefix blocks)
    const int seq_tok0 = bi.k_tok0;      // K/V tokens of the sequence: seq_tok0 .. last_tok
    const int last_tok = bi.k_end - 1;

    const int tid = threadIdx.x, l = tid & 63, half = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index, held in a scalar register
    const int q_local = 32 * w + (l & 31);
    const int qoff = 128 * sub;                               // the workgroup's first query within the q-block
    const int q_len = bi.q_len - qoff < 128 ? bi.q_len - qoff : 128;   // its valid queries
    if (q_len <= 0) return;                                   // a ragged q-block that ends before this part
    const int q_tok0 = bi.q_tok0 + qoff;

    // The first two list entries are fetched together with the count (the memory is there whatever
    // the count says), so that the first tile loads do not wait for a second round trip.
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
    // Tiles: TPB per listed block.  Of the diagonal block (only the last entry can be it) this part
    // of the q-block needs the tiles up to its own last query, 2 (sub + 1) of them; that is fewer than
    // TPB only for the first half of a 256-query block.  The count is even in every case.
    int ntiles = TPB * nb;
    if (TPB > 2 && nb > 0 && 2 * (sub + 1) < TPB) {
        const int bl = SPARSE ? list[nb - 1] : nb - 1;
        if (bl >= I) ntiles -= TPB - 2 * (sub + 1);
    }

    if (ntiles == 0) {   // empty list: O = 0, lse = -inf (uniform exit, before any barrier)
        if (q_local < q_len) {
            uint16_t *op = O + ((size_t)(q_tok0 + q_local) * hq + h) * D + (D / 2) * half;
            const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < D / 16; ++i) *reinterpret_cast<u32x4 *>(op + 8 * i) = z;
            if (lse != nullptr && half == 0) lse[(size_t)h * T + q_tok0 + q_local] = -INFINITY;
        }
        return;
    }

#define FP_TILE_BLOCK(t) attn_tile_block<SPARSE, TPB>(list, (t), I, nb)

    // Q^T B-fragments: query 32w + l%32, dims 16ks + 8*half..+7.  The loads are written as
    // assembly so that their completion is counted here and not by the compiler, which cannot see
    // the tile loads queued behind them and would wait for those too: the prologue waits once,
    // with the exact count, for the fragments and the first K tile together.
    bf16x8 qb[KS];
    {
        int row = q_local < q_len ? q_local : q_len - 1;
        const uint16_t *qp = Q + ((size_t)(q_tok0 + row) * hq + h) * D + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (kAttnAgpr<D>) asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=&a"(qb[ks]) : "v"(qp), "n"(32 * ks) : "memory");
            else asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=&v"(qb[ks]) : "v"(qp), "n"(32 * ks) : "memory");
        }
    }

    // Tile loads.  One wave-wide instruction moves RPL = 512/D rows (1 KB); wave w loads rows
    // 16w + RPL i + l/LPR (i < LPT) of a K or V tile (head dimension 128: 4 rows per instruction,
    // rows 16w + 4i + l/16).  Lane l fills LDS position l % LPR of its row, i.e. it fetches the
    // global chunk (l % LPR) ^ swizzle(row).  The global address is a wave-uniform base (first token
    // of the tile, KV head) plus a per-lane 32-bit byte offset.  Only a tile that reaches past
    // the end of its sequence (ragged last block) needs per-row clamping; its base is clamped
    // too, so the unsigned row offsets can never wrap.
    const uint32_t row_bytes = (uint32_t)hkv * D * 2;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(FP_LDS(char) *)smem;
    const uint32_t ld_dst = __builtin_amdgcn_readfirstlane(lds_base + 16 * w * RB);
    const int ld_row = 16 * w + l / LPR;   // + RPL i
    const int ld_pos = l % LPR;
    const char *Kb = reinterpret_cast<const char *>(K) + (size_t)hk * D * 2;
    const char *Vb = reinterpret_cast<const char *>(V) + (size_t)hk * D * 2;
    uint32_t ld_kcol[LPT], ld_vcol[LPT];   // byte offset from the tile's first row; see kAttnRowInOffset
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int row = ld_row + RPL * i, off_row = kAttnRowInOffset<D> ? row : ld_row;
        ld_kcol[i] = (uint32_t)((ld_pos ^ swz<D>(row)) * 16) + (uint32_t)off_row * row_bytes;
        ld_vcol[i] = (uint32_t)((ld_pos ^ (4 * attn_vswz<D>(row))) * 16) + (uint32_t)off_row * row_bytes;
    }
    // Clamped load of sub-tile sub_ of block blk_: every row is kept at or before the sequence's last token.
#define FP_LOAD(Xb, col_, blk_, sub_, ldsoff_)                                                            \
    do {                                                                                                  \
        const int tok0_ = seq_tok0 + (blk_) * BLK + (sub_) * KT;                                          \
        const int base_tok_ = tok0_ < last_tok ? tok0_ : last_tok;                                        \
        const char *base_ = Xb + (size_t)base_tok_ * row_bytes;                                           \
        const uint32_t dst_ = __builtin_amdgcn_readfirstlane(ld_dst + (ldsoff_));                                         \
        _Pragma("unroll") for (int i_ = 0; i_ < LPT; ++i_) {                                              \
            int tok_ = tok0_ + ld_row + RPL * i_;                                                         \
            tok_ = tok_ < last_tok ? tok_ : last_tok; /* keys past the end are masked as future */        \
            const uint32_t ro_ = (uint32_t)(tok_ - base_tok_) * row_bytes; /* tok_ >= base_tok_ */        \
            load_to_lds(base_, ro_ + (col_[i_] - (uint32_t)(ld_row + (kAttnRowInOffset<D> ? RPL * i_ : 0)) * row_bytes), dst_ + i_ * 1024); \
        }                                                                                                 \
    } while (0)
    // Tile t lives in K and V buffer t % 2.
#define FP_KBUF(par) ((uint32_t)((par) * kAttnTile<D, KT>))
#define FP_VBUF(par) ((uint32_t)(kAttnVBase<D, KT> + (par) * kAttnTile<D, KT>))
    // Offset of tile u given its list entry; the block id is kept inside the blocks that are complete
    // in memory (those before the diagonal one, and the diagonal one unless the sequence ends inside
    // it), so that even a malformed (non-ascending) list cannot make a plain load reach past the sequence.
    const bool diag_full = seq_tok0 + (I + 1) * BLK - 1 <= last_tok;
    const int ent_max = diag_full ? I : I - 1;
#define FP_ENT_OFF(ent_, u)                                                                               \
    ((uint64_t)(uint32_t)(seq_tok0 + ((ent_) < 0 ? 0 : ((ent_) < ent_max ? (ent_) : ent_max)) * BLK + ((u) % TPB) * KT) * row_bytes)

    f32x16 acc[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float m_run = -INFINITY;   // reference point of the exponentials (raw dot-product units), see attn_new_max
    float l_run = 0.f;         // this lane's share of the running row sum

    // Fragment addresses inside a buffer.  K: rows l%32 and 32 + l%32, chunk
    // (2ks + half) ^ swz(row) = 2ks ^ (half ^ swz(row)); rows 32 apart share the permutation.
    const int krow = l & 31;
    const uint32_t k_frag = (uint32_t)(krow * RB + ((half ^ swz<D>(krow)) << 4));
    // V transpose reads: row 32kt + 16j + 4half + e (+8), e = (l%16)/4 = row & 3; 8-byte unit at
    // dims 32dt + 16gq + 4cc, i.e. chunk 4dt + 2gq + cc/2, stored at chunk ^ 4 vswz(e)
    // = 4(dt ^ vswz(e)) + ...
    uint32_t v_frag[NDT];
    {
        const int e = (l & 15) >> 2, gq = (l & 31) >> 4, cc = l & 3;
        const uint32_t vb = (uint32_t)((4 * half + e) * RB + (2 * gq + (cc >> 1)) * 16 + 8 * (cc & 1));
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) v_frag[dt] = vb + (uint32_t)((dt ^ attn_vswz<D>(e)) * 64);
    }
    // Causal limit of tile t for this lane: on the diagonal block, key kk of the tile is in the
    // lane's future if kk > query - tile offset (and keys past a ragged end lie beyond every stored
    // query); elsewhere nothing is masked.
#define FP_LIM(t) (FP_TILE_BLOCK(t) == I ? qoff + q_local - ((t) % TPB) * KT - 4 * half : 2 * KT)

    // Prologue: S^T of tile 0 with its row max; on leaving it K[1] and V[0] are in and the first
    // fragments of K[1] are being read.
    FP_LOAD(Kb, ld_kcol, b0, 0, FP_KBUF(0));
    FP_LOAD(Kb, ld_kcol, b0, 1, FP_KBUF(1));   // ntiles >= 2
    FP_LOAD(Vb, ld_vcol, b0, 0, FP_VBUF(0));
    FP_WAIT_VMCNT(2 * LPT);   // Q and K[0] are in; K[1] and V[0] keep landing under the first QK^T
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {   // uses of Q stay behind the wait
        if constexpr (kAttnAgpr<D>) asm volatile("" : "+a"(qb[ks]));
        else asm volatile("" : "+v"(qb[ks]));
    }
    __syncthreads();
    constexpr int NKT = KT / 32;
    f32x16 sA[NKT], sB[NKT];
    bf16x8 ring[kAttnRing];
    static_for<NKT * KS>([&](auto f_) __attribute__((always_inline)) {
        constexpr int f = f_;
        attn_mfma_s<D, (f < NKT)>(sA[f % NKT], attn_kfrag<D, KT>(smem, FP_KBUF(0) + k_frag, f), qb[f / NKT]);
    });
    attn_settle<D, KT>(sA);
    attn_mask<KT>(sA, b0 == I ? qoff + q_local - 4 * half : 2 * KT);
    m_run = halves_max(attn_rowmax_half<KT>(sA));   // finite: key 0 of tile 0 is visible to every query
    FP_WAIT_VMCNT(0);
    __syncthreads();
#pragma unroll
    for (int f = 0; f < kAttnRing - 1; ++f) ring[f] = attn_kfrag<D, KT>(smem, FP_KBUF(1) + k_frag, f);

    // Step t (attn_step) loads K[t+2] and V[t+1].  Variants:
    //   MAIN  tile t+1 needs no mask, tiles t+1 and t+2 are complete in memory: cheap loads;
    //   TAIL  row-clamped loads and the (branch-free) causal limit of tile t+1;
    //   PEN   the last but one step: as TAIL without a K load or the reads of a next K tile;
    // the last tile's exponentials and PV follow the loops.  PAR is the parity of t (steps come in pairs
    // that start at an even t): tiles t live in K and V buffers PAR.
    // A tile of the diagonal block that lies wholly in a wave's future needs no special case: its
    // logits are all -inf, which leaves the max alone and contributes zeros.
#define FP_STEP(MODE, PAR, t, sc, sn, LOADX)                                                               \
    do {                                                                                                  \
        const int t_ = (t);                                                                               \
        uint32_t va_[NDT];                                                                                \
        _Pragma("unroll") for (int dt_ = 0; dt_ < NDT; ++dt_) va_[dt_] = FP_VBUF(PAR) + v_frag[dt_];      \
        attn_step<D, KT, MODE>(                                                                           \
            smem, FP_KBUF(1 - PAR) + k_frag, FP_KBUF(PAR) + k_frag, va_, qb, sc, sn, acc, m_run, l_run, ring, c, LOADX, \
            [&]() __attribute__((always_inline)) { FP_WAIT_VMCNT(0); __syncthreads(); },                  \
            [&]() __attribute__((always_inline)) { attn_settle<D, KT>(sn); attn_mask<KT>(sn, FP_LIM(t_ + 1)); }); \
    } while (0)
    // load i of a step, K first; VOFF / KOFF are the byte offsets of tiles t+1 / t+2
#define FP_LOAD_MAIN(PAR, VOFF, KOFF)                                                                      \
    [&](int i_) __attribute__((always_inline)) {                                                          \
        const bool k_ = i_ < LPT;                                                                         \
        const int j_ = k_ ? i_ : i_ - LPT;                                                                \
        const char *base_ = k_ ? Kb + (KOFF) : Vb + (VOFF);                                               \
        const uint32_t col_ = k_ ? ld_kcol[j_] : ld_vcol[j_];                                             \
        const uint32_t dst_ = ld_dst + (k_ ? FP_KBUF(PAR) : FP_VBUF(1 - (PAR))) + j_ * 1024;              \
        if constexpr (kAttnRowInOffset<D>) load_to_lds(base_, col_, dst_);                                \
        else load_to_lds_add(base_, (uint32_t)(RPL * j_) * row_bytes, col_, dst_);                        \
    }
#define FP_LOAD_TAIL(PAR, t, WITH_K)                                                                       \
    [&](int i_) __attribute__((always_inline)) {                                                          \
        if (i_ == 0 && WITH_K) FP_LOAD(Kb, ld_kcol, FP_TILE_BLOCK((t) + 2), (((t) + 2) % TPB), FP_KBUF(PAR)); \
        if (i_ == LPT) FP_LOAD(Vb, ld_vcol, FP_TILE_BLOCK((t) + 1), (((t) + 1) % TPB), FP_VBUF(1 - (PAR))); \
    }

    // Tiles before the diagonal block are complete (only a sequence's last block can be partial,
    // and a row only meets it as its diagonal); the list is ascending, so only its last block can
    // be the diagonal one: the first n_plain tiles need no mask.  A pair of MAIN steps (t, t+1)
    // computes S^T of tiles t+1 and t+2 without a mask and loads tiles up to t+3 without a clamp;
    // ntiles and n_plain are even, so t < n_plain - 2 gives t+3 < n_plain.  Steps come in pairs, so
    // the register roles of the two S^T tiles alternate evenly.
    const int n_plain = FP_TILE_BLOCK(ntiles - 1) == I ? TPB * (nb - 1) : ntiles;
    const int t_main = n_plain - 2;   // <= 0: none
    int t = 0;
    if (t_main > 0) {
        // Addresses of the main loop, carried instead of recomputed: o1..o3 = offsets of tiles t+1..t+3,
        // e2 = list entry of tile t+2, fetched one pair of steps before it is needed (a list read is a
        // scalar memory load; waiting for it inside a step would stall the wave).  Tile t+3 is the odd
        // neighbour of t+2 in one block.  (Tiles 0..2 lie in the first two list entries at most.)
        uint64_t o1 = FP_ENT_OFF(b0, 1);
        int e2 = 2 / TPB == 0 ? b0 : b1;
        for (; t < t_main; t += 2) {
            const uint64_t o2 = FP_ENT_OFF(e2, t + 2);
            const uint64_t o3 = o2 + (uint64_t)KT * row_bytes;
            const int u4 = (t + 4) / TPB < nb ? (t + 4) / TPB : nb - 1;
            e2 = SPARSE ? list[u4] : u4;
            FP_STEP(MAIN, 0, t, sA, sB, FP_LOAD_MAIN(0, o1, o2));
            FP_STEP(MAIN, 1, t + 1, sB, sA, FP_LOAD_MAIN(1, o2, o3));
            o1 = o3;
        }
    }
    for (; t < ntiles - 2; t += 2) {
        FP_STEP(TAIL, 0, t, sA, sB, FP_LOAD_TAIL(0, t, true));
        FP_STEP(TAIL, 1, t + 1, sB, sA, FP_LOAD_TAIL(1, t + 1, true));
    }
    FP_STEP(PEN, 0, t, sA, sB, FP_LOAD_TAIL(0, t, false));
    {
        bf16x8 pb[KT / 16];
        float x[KT / 2], ls[NKT];
        attn_exp<KT, 0, KT / 2>(sB, c, m_run * c, x);
        attn_exp_done<KT, 0, KT / 2>(x, ls, pb);
        l_run += attn_tile_sum<KT>(ls);
        uint32_t va[NDT];
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) va[dt] = FP_VBUF(1) + v_frag[dt];
#pragma unroll
        for (int v = 0; v < KT / 16 * NDT; ++v) acc[v % NDT] = mfma32(attn_vfrag<D>(smem, va, v), pb[v / NDT], acc[v % NDT]);
    }

    // O = acc / l, lse = m + log2 l (Alg. 3, final normalisation); rows past a ragged end are not stored.
    // Each lane holds 4 consecutive dims of one query per accumulator group, which would make every
    // global store touch 64 different rows.  The wave's 32 x D output tile is therefore turned
    // through LDS (its own 32 rows of the K buffers: their last reader and their last incoming load
    // finished before the barrier of the last-but-one step) into 16-byte pieces, D/8 lanes per row.
    // Chunk c of row q is kept at chunk c ^ swz(q) so that neither side meets a bank conflict.
    const float l_tot = halves_sum(l_run);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    {
        char *ob = smem + w * (32 * RB);
        const int qrow = l & 31;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[dt][4 * q4 + e] * inv);
                *reinterpret_cast<bf16x4 *>(ob + qrow * RB + (((4 * dt + q4) ^ swz<D>(qrow)) << 4) + 8 * half) = o;
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int lo = l;   // opaque, so that the row of each store is not computed ahead and carried through the loop: no register is left at
        asm volatile("" : "+v"(lo));   // head dimension 64 (one was spilled: 8 bytes of scratch)
        const int pc = lo % LPR;
#pragma unroll
        for (int i = 0; i < 32 / RPL; ++i) {
            const int orow = RPL * i + lo / LPR;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(ob + orow * RB + (pc << 4));
            if (32 * w + orow < q_len)
                *reinterpret_cast<u32x4 *>(O + ((size_t)(q_tok0 + 32 * w + orow) * hq + h) * D + ((pc ^ swz<D>(orow)) << 3)) = v;
        }
    }
    if (q_local < q_len && lse != nullptr && half == 0)
        lse[(size_t)h * T + q_tok0 + q_local] = l_tot > 0.f ? m_run * c + __log2f(l_tot) : -INFINITY;
#undef FP_TILE_BLOCK
#undef FP_LOAD
#undef FP_LOAD_MAIN
#undef FP_LOAD_TAIL
#undef FP_ENT_OFF
#undef FP_LIM
#undef FP_KBUF
#undef FP_VBUF
#undef FP_STEP
}

}  // namespace fp
