// Shared device-side definitions for the gfx950 kernels (wave64, bf16 MFMA, 160 KB LDS).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace fp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The kernels are templates over the head dimension D (64, 128 or 256).  A row of D bf16 is
// D/8 16-byte chunks; LDS tiles are unpadded and keep chunk c of row r at position c ^ swz<D>(r)
// (see the kernels).
template <int D> constexpr int kChunks = D / 8;                            // 16-byte chunks per row
// Chunk permutation of row r: 16 consecutive rows at one chunk lie in 16 different bank groups of 16 bytes (the banks are 256
// bytes wide: one row of D = 128, two of 64).
template <int D> __device__ __forceinline__ constexpr int swz(int r) { return D < 128 ? (r >> 1) & (kChunks<D> - 1) : r & 15; }
template <int D> constexpr int kRowsPerLoad = 512 / D;                     // rows one 1 KB wave-wide load covers
// Key blocks of a sequence (512K tokens in blocks of 128).  The search keeps one float per block and head of a row in LDS beside its
// tile buffers, which would allow more, and its candidates as 64 bits per lane, which would not.
constexpr int kMaxBlocksPerSeq = 4096;
constexpr float kLog2e = 1.4426950408889634f;

// One q-block row.  Queries: first token of the block (index into Q and O) and the number of
// valid tokens in it (1..128).  I = the block's index within its sequence, i.e. its index within
// the query chunk plus the KV prefix in blocks; its causal key blocks are J <= I.  Keys: the
// sequence's first token (index into K and V), one past its last, the first row of its pooled
// keys in the workspace and the number of its key blocks.
struct __attribute__((aligned(16))) RowRec {
    int q_tok0, q_len, I, kb_row0;
    int k_tok0, k_end, n_kb, pad1;
};
// One key block: first token and number of valid tokens.
typedef int2 KeyBlockRec;

// f(0), f(1) .. f(N-1) with the index as a compile-time constant.
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

#define FP_LDS(T) __attribute__((address_space(3))) T

__device__ __forceinline__ float bf16lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// v_mfma_f32_32x32x16_bf16: A is 32x16 (lane l holds row l%32, k = 8*(l/32)..+7), B is 16x32
// (lane l holds column l%32, same k), the 32x32 result keeps column l%32 in lane l and row
// 8*(r/4) + 4*(l/32) + r%4 in register r.
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Combine each lane's value with that of lane l ^ 32 through the register swap between the two
// halves of the wave (v_permlane32_swap exchanges the upper half of its first operand with the
// lower half of its second): applied to two copies of x, one register ends up with x[l % 32] and
// the other with x[32 + l % 32] in every lane.  Unlike a shuffle through the LDS crossbar this
// leaves the LDS queue alone, so no wait on outstanding fragment reads is needed around it.
// Written as inline assembly because the compiler's builtin folds the two results into one when
// both inputs are the same value; the s_nop covers the wait states the instruction needs after
// a VALU write of its operands.
__device__ __forceinline__ void halves_swap(float x, float &lo, float &hi) {
    lo = x;
    hi = x;
    asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
}
__device__ __forceinline__ float halves_max(float x) {
    float a, b;
    halves_swap(x, a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float halves_sum(float x) {
    float a, b;
    halves_swap(x, a, b);
    return a + b;
}

// The same between lanes l and l ^ 16: v_permlane16_swap exchanges the odd rows of 16 lanes of its first operand with the
// even ones of its second.
__device__ __forceinline__ void rows_swap(float x, float &even, float &odd) {
    even = x;
    odd = x;
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(even), "+v"(odd));
}
// x of the lane N places further round its row of 16.
template <int N> __device__ __forceinline__ float row_turn(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x120 + N, 0xf, 0xf, true));
}

// Over the whole wave, result in every lane: halves, rows, then turns by 8, 4, 2 and 1 inside a row.  After a turn by n all
// values repeat every n lanes, so that the next one meets the lane an exchange l ^ n/2 would meet: the sums are those of a
// butterfly, bit for bit.  All six stages stay in registers; through the LDS crossbar (__shfl_xor) each was a round
// trip of its own, and a row of the search goes through up to eight such reductions one after another (pooling and one-pass
// search, 8K tokens: 26.1 -> 23.2 us, a 2000-token chunk 54.5 -> 52.6, head dimension 64 at 16K 28.0 -> 26.1).
__device__ __forceinline__ float wave_max(float v) {
    float a, b;
    rows_swap(halves_max(v), a, b);
    v = fmaxf(a, b);
    v = fmaxf(v, row_turn<8>(v));
    v = fmaxf(v, row_turn<4>(v));
    v = fmaxf(v, row_turn<2>(v));
    return fmaxf(v, row_turn<1>(v));
}
__device__ __forceinline__ float wave_sum(float v) {
    float a, b;
    rows_swap(halves_sum(v), a, b);
    v = a + b;
    v += row_turn<8>(v);
    v += row_turn<4>(v);
    v += row_turn<2>(v);
    return v + row_turn<1>(v);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max of three.  The device code is compiled with NaNs not honoured (see build.py), so this
// becomes one v_max3_f32 instead of three canonicalising v_max_f32 plus the max itself.  It must
// stay a compiler-visible instruction: the wait states the hardware needs between an MFMA and a
// VALU read of its result are inserted by the compiler, and inline assembly would not get them.
// (The attention kernel's exponentials are assembly and read MFMA results all the same: each of them has
// gone through a max3 before.  Results of MFMAs that are themselves assembly get no wait states here either.)
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// 16 bytes per lane, global -> LDS, no register staging: lane i's 16 bytes, fetched from
// sbase + voff, land at LDS byte address lds_addr + 16 i (lds_addr is wave-uniform and goes to
// M0).  Written as inline assembly on purpose: the compiler then neither tracks these loads in
// vmcnt nor orders LDS reads after them (it would wait for *all* outstanding loads before the
// first LDS read of every step, which defeats the prefetch).  Completion is waited for
// explicitly with FP_WAIT_VMCNT followed by a workgroup barrier.
// M0 is named as clobbered so that the compiler does not keep a value of its own in it across
// the statement; it answers with a warning that it will not save and restore a reserved register
// for us, which is what is wanted here (no code in these kernels needs M0 otherwise).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(const char *sbase, uint32_t voff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(sbase), "s"(lds_addr)
                 : "memory", "m0");
}
// The same with the lane's offset as the sum of a wave-uniform and a per-lane part: the addition fills
// the wait state the load needs after the write of M0.
__device__ __forceinline__ void load_to_lds_add(const char *sbase, uint32_t soff, uint32_t voff, uint32_t lds_addr) {
    uint32_t at;
    asm volatile("s_mov_b32 m0, %4\n\tv_add_u32 %0, %1, %2\n\tglobal_load_lds_dwordx4 %0, %3"
                 : "=&v"(at)
                 : "s"(soff), "v"(voff), "s"(sbase), "s"(lds_addr)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// s_waitcnt vmcnt(n) alone (expcnt and lgkmcnt left at "no wait"), n < 64: the count's low four
// bits sit in bits 3:0 of the immediate, its high two in bits 15:14
#define FP_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0f70 | ((n) & 15) | (((n) >> 4) << 14))

}  // namespace fp
