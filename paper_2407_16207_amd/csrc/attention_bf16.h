// What the two bf16 attention kernels (dag_attention_bf16.hip, dag_attention_bf16_keys.hip) share: parameters, operand
// types, global -> LDS copies; and the merge of split partials, which the fp32 kernel uses too.
#pragma once
#include "gsd_internal.h"

namespace gsd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMInit = -1e30f;     // finite stand-in for -inf: the offset stored for a partial without any visible key

struct AttnParams {
    const __bf16 *q;
    __bf16 *o;
    float *lse;
    const __bf16 *k;
    const __bf16 *v;
    const int64_t *kv_offsets;
    const int32_t *prefix_lens;
    const int32_t *node_offsets;
    const uint64_t *mask;
    float *part_o;      // [splits][T][Hq][D] fp32 unnormalised
    float *part_ml;     // [splits][T][Hq][2]  (offset in the log2 domain, sum of 2^(score - offset))
    int64_t q_ts, q_hs, o_ts, o_hs, kv_ts, kv_hs;
    int32_t batch, total_nodes, max_nodes, num_q_heads, num_kv_heads, group, words_per_row;
    int32_t q_tiles;    // row tiles per (sequence, KV head)
    int32_t splits;
    int32_t wg_per_xcd; // ceil(batch * num_kv_heads / 8) * q_tiles * splits
    float scale_log2e;  // softmax_scale * log2(e)
};

// position of actual key row r (0..63) inside the LDS K tile: bits 2 and 3 of r swapped (an involution)
__device__ __forceinline__ int k_lds_row(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

// max over the two 32-lane halves of a wavefront, in every lane
__device__ __forceinline__ float max_across_halves(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// One 16-byte-per-lane global -> LDS copy: lane l's 16 bytes at gbase + voff land at LDS byte lds_base + 16*l.
// Issued as inline assembly so that the compiler's wait-count pass does not serialise later LDS reads behind
// it; completion is awaited by hand (dma_wait) before the barrier that publishes the tile.
__device__ __forceinline__ void dma16(const void *gbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                 :: "s"(gbase), "v"(voff), "s"(lds_base) : "memory");
}
// The same with the LDS address as a scalar base plus a constant, added inside: given one scalar per destination
// the compiler keeps them all live across the loop (sixteen at four copies per tile and wave) and spills them.
__device__ __forceinline__ void dma16_at(const void *gbase, uint32_t voff, uint32_t lds_base, int lds_const) {
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                 :: "s"(gbase), "v"(voff), "s"(lds_base), "i"(lds_const) : "memory", "scc");
}
// From any address per lane, 16 or 4 bytes of it; lane l's land at lds_base + 16*l or + 4*l.
__device__ __forceinline__ void dma16_from(const void *at, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(at), "s"(lds_base) : "memory");
}
__device__ __forceinline__ void dma4_from(const void *at, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" :: "v"(at), "s"(lds_base) : "memory");
}
template <int N> __device__ __forceinline__ void dma_wait() {   // at most N vector-memory operations in flight
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// A wave-uniform 64-bit value, forced into scalar registers (the copies above take their base address from there;
// a uniform value loaded through the vector memory path would otherwise stay in vector registers).
__device__ __forceinline__ int64_t uniform64(int64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(x)));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(uint64_t(x) >> 32));
    return int64_t((uint64_t(hi) << 32) | lo);
}
// Work-group barrier as bare assembly: the compiler's own barrier is preceded by a wait for every outstanding LDS
// read, which would undo the reads issued ahead of it on purpose (their results are awaited where they are used).
__device__ __forceinline__ void wg_barrier() {
    asm volatile("s_barrier" ::: "memory");
}

// Matrix instructions written out for one wavefront per SIMD.  With 512 registers per lane the compiler
// selects the accumulator-register form for every matrix instruction it emits itself, and then moves every score
// into an ordinary register before the softmax can touch it.  Written out, the score accumulators stay in ordinary
// registers ("v") and only the output accumulators and the query fragments, which the vector ALU never reads in
// the loop, live in accumulator registers ("a").  The compiler does not know these are matrix instructions, so
// the two places where the vector ALU reads their results soon after them wait by hand (mfma_settle).
__device__ __forceinline__ void mfma_v_acc(floatx16 &acc, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_v_init(floatx16 &acc, const bf16x8 &a, const bf16x8 &b) {   // starts a chain from zero
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=v"(acc) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_a_acc(floatx16 &acc, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// at least 16 issue cycles: longer than the 12 the vector ALU must keep away from an 8-pass matrix result
__device__ __forceinline__ void mfma_settle() { asm volatile("s_nop 7\n\ts_nop 7" ::: "memory"); }

hipError_t launch_attention_combine(const AttnParams &p, int head_dim, int dtype, hipStream_t stream);
hipError_t launch_attention_bf16_keys(const AttnParams &p, int head_dim, int row_groups, hipStream_t stream);

}  // namespace gsd
