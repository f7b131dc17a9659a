// What the bf16 attention kernels share: the launch parameters, the MFMA operand helpers, the direct
// global -> LDS loads and the layout of the partial results of a launch that splits the key axis.
#pragma once

#include <math.h>
#include <type_traits>

#include "kvcomm_device.h"

namespace kvc {

struct AttnParams {
    const void *q, *k, *v;
    void *out;
    float *lse;
    Strides s_q, s_k, s_v, s_o;
    int32_t L, Hkv, G, n_ctx, tq, N;
    int32_t n_row_tiles;
    int32_t n_items;   // L * Hkv * n_row_tiles (* n_splits)
    float scale;       // softmax scale
    float scale_log2;  // scale * log2(e)
    // Split launches: the keys of a row tile are cut into n_splits runs of 64-key tiles (split_bound below) and
    // every (row group, split) leaves its unnormalised output, reference and row sum here.
    float *part_o;     // [group][split][D / 4 slots of 4 channels x rows of a group], see part_slot
    float *part_ml;    // [group][split][2][rows of a group]: reference m (raw score units), row sum
    int32_t n_splits;  // 1: results go straight to `out`
    int32_t groups_per_tile;  // groups of a row tile: bf16, of 32 rows (= wavefronts that own rows; one of 16 in a tile of 16 rows); fp32, of 16
    divisor_t by_G, by_Hkv, by_row_tiles, by_splits, by_groups;   // set_divisors()
};
__device__ __forceinline__ void await_attn_args(const AttnParams &p)
{
    await_args(arg_word(&p), arg_word(&p.s_q.token), arg_word(&p.s_v), arg_word(&p.L));
    await_args(arg_word(&p.n_splits), arg_word(&p.by_groups));
}
static inline void set_divisors(AttnParams &p)
{
    p.by_G = make_divisor((uint32_t)p.G);
    p.by_Hkv = make_divisor((uint32_t)p.Hkv);
    p.by_row_tiles = make_divisor((uint32_t)p.n_row_tiles);
    p.by_splits = make_divisor((uint32_t)p.n_splits);
    p.by_groups = make_divisor((uint32_t)p.groups_per_tile);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef short s16x4 __attribute__((ext_vector_type(4)));

// Two 8-byte transposing LDS reads (ds_read_b64_tr_b16) -> one 8 x bf16 MFMA operand.
// Within each group of 16 lanes the instruction returns to lane i, element e, the 16-bit
// element (i % 4) found at the address supplied by lane 4*e + i/4 of the group.
__device__ __forceinline__ bf16x8 lds_read_tr_pair(const lds_byte *a0, const lds_byte *a1)
{
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a0);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a1);
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// One wavefront-wide direct load global -> LDS (global_load_lds_dwordx4): lane i moves the 16 bytes at
// global address `base` + `voff` (a wavefront-uniform 64-bit base in scalar registers plus its own unsigned
// 32-bit byte offset) to LDS address `dst` + 16 * i (`dst` is wavefront-uniform and travels in M0).
// Written as inline assembly on purpose: the compiler then does not know of the pending LDS write and
// inserts no wait of its own before later LDS reads (it would wait for ALL outstanding loads ahead of the
// first transposing read and so serialise the prefetch).  Ordering is explicit instead: the kernels wait for
// the loads (vmcnt) and, where another wavefront reads what they wrote, synchronise the block.
// M0 is listed as clobbered, so the compiler re-forms it for any instruction of its own that needs it.
// (clang warns about any reserved register in a clobber list; for M0, which it only ever sets immediately
// before the instruction that reads it, the declaration is exactly what is meant.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool NT = false>   // NT: non-temporal (data that nobody reads again)
__device__ __forceinline__ void dma16_sbase(const unsigned char *base, uint32_t voff, const lds_byte *dst)
{
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(voff), "s"(base), "s"(m0) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base), "s"(m0) : "memory", "m0");
}

template <int V>
using template_int = std::integral_constant<int, V>;

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// The same with the LDS destination as a wavefront-uniform base plus a literal (M0 is formed by one scalar
// add): the steady-state loads then cost no vector ALU instruction and no register per destination (the
// row base advances on the scalar unit and the per-lane offset never changes).
template <int OFF>
__device__ __forceinline__ void dma16_sbase_at(const unsigned char *base, uint32_t voff, uint32_t dst_base)
{
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 : : "v"(voff), "s"(base), "s"(dst_base), "n"(OFF) : "memory", "scc", "m0");
}
#pragma clang diagnostic pop

// ------------------------------------------------------------------------------ split key axis
// First unit (64-key tile or 32-key sub-step) of split s of a row tile whose queries see keys [0, n_ctx + imax]
// (`units` of them in all).  Every split starts at a key that all queries of the tile see (`first_hidden` =
// units from which that no longer holds, i.e. floor((n_ctx + imin) / unit) + 1): the causal edge belongs to the
// last split that is not empty.  Splits beyond that are empty (bound(s) == bound(s + 1)) and leave reference -inf.
__host__ __device__ __forceinline__ int split_bound(int s, int n_splits, int units, int first_hidden)
{
    if (s >= n_splits) return units;
    const int b = s * units / n_splits;   // n_splits <= 16, units <= 2^26: no overflow
    return b < first_hidden ? b : (s == 0 ? 0 : units);
}

// Output accumulators of a 32-row group (attn_rows_kernel16: of 16, likewise) travel as 16-byte slots: slot (c4, n) = channels 4 * c4 ... + 3 of row n, rows
// fastest, as the MFMAs leave them (256- and 512-byte runs).
__device__ __forceinline__ int part_slot(int c4, int n) { return c4 * 32 + n; }

// acc = A B and acc += A B, the accumulator in place (ACC: in the accumulation registers).  Through the builtin the compiler gives
// the sum other registers than the addend and hands the addend's to the vector instructions that follow, each of which
// then waits for the MFMA.  It inserts no wait states around inline assembly: no vector instruction may write an operand in the
// two wait states before it (kGuarded waits for those itself) or touch `acc` in the eight after it (mfma_settle waits that long).
// tests/test_mfma_hazards.py looks for such instructions in the built library.
enum class Mfma { kBuiltin, kInPlace, kGuarded };

template <Mfma HOW>
__device__ __forceinline__ void mfma_first(f32x4 &acc, const bf16x8 a, const bf16x8 b)
{
    if constexpr (HOW == Mfma::kBuiltin)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    else if constexpr (HOW == Mfma::kInPlace)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
    else
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}
template <Mfma HOW, bool ACC = false>
__device__ __forceinline__ void mfma_next(f32x4 &acc, const bf16x8 a, const bf16x8 b)
{
    if constexpr (HOW == Mfma::kBuiltin)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    else if constexpr (HOW == Mfma::kInPlace && !ACC)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
    else if constexpr (HOW == Mfma::kInPlace)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    else if constexpr (!ACC)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
    else
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
template <bool ACC, int N>
__device__ __forceinline__ void mfma_settle(f32x4 (&o)[2][N])
{
    asm volatile("s_nop 7\n\ts_nop 7" : : : "memory");
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if constexpr (ACC)
            asm volatile("" : "+a"(o[0][i]), "+a"(o[1][i]));
        else
            asm volatile("" : "+v"(o[0][i]), "+v"(o[1][i]));
    }
}

// 16x16x32 MFMAs leave a query column in the four lanes n, 16 + n, 32 + n, 48 + n: their maximum and their sum.
__device__ __forceinline__ float query_max(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float query_sum(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace kvc
