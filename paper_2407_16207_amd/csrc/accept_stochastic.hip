// Non-deterministic verification (paper Section 3: the i-th drafted token is accepted with probability
// min(1, p/q), the first rejection discards the rest of the hypothesis and the LLM regenerates that token;
// Section 6.4: the setting on token graphs).  Two kernels:
//
//   softmax_stats_kernel    one pass over a logits row: running (max, sum of exp(x - max)) per lane, merged across
//                           the work-group: the normaliser of the LLM's distribution after every node.  HBM-bound,
//                           same traffic as the argmax pass of deterministic verification.
//   accept_and_resample_kernel one work-group per sequence, in two phases that share everything but the vocabulary rows:
//     accept_phase            every edge r -> i is tested once,
//                               accept_u[i] * draft_prob[i] < p_r(token_i)      (<=> u < min(1, p/q) for u < 1)
//                           with p_r(token_i) = exp(logit - max_r) / sum_r gathered from the row of r, then the same
//                           relaxation, end-node choice and back-walk as the deterministic kernel.
//     resample_phase          the regenerated token, drawn by inverse CDF from max(p - q, 0) at the end of the accepted
//                           path (from p if that node has no children or the residual is empty).  Every thread owns a
//                           contiguous slice of the vocabulary, slice sums are scanned in thread order, the owning
//                           thread walks its slice: one fixed summation order.
//                           (resample_held_phase: the same with the slices kept in registers, where they fit.)
// Both phases are chains of dependent round trips on one CU per sequence.  As two kernels (7.0 + 11.7 us on 8 sequences
// of 256 nodes, 32000 tokens) the second waited for a launch and fetched end node, offsets and parents again: together
// 16.7 us, now 14.6.  What is left is mostly the vector work of one CU: exponentials of 32000 draft logits 2.2 us, weights 3.5.
// With more sequences than CUs they are two kernels all the same (accept_stochastic_kernel, resample_kernel).
#include <type_traits>

#include "gsd_internal.h"

namespace gsd {

__device__ __forceinline__ float load_logit(const void *base, int64_t elem, int dtype) {
    if (dtype == GSD_BF16) return __uint_as_float(uint32_t(reinterpret_cast<const uint16_t *>(base)[elem]) << 16);
    return reinterpret_cast<const float *>(base)[elem];
}

// (m, s) <- merge of two partial softmax states: s counts exp(x - m)
__device__ __forceinline__ void merge_state(float &m, float &s, float m2, float s2) {
    const float mm = fmaxf(m, m2);
    if (mm == -__builtin_inff()) {          // both empty (or all -inf so far)
        m = mm;
        s = 0.f;
        return;
    }
    s = s * __expf(m - mm) + s2 * __expf(m2 - mm);
    m = mm;
}

template <int THREADS, bool BF16>
__global__ __launch_bounds__(THREADS) void softmax_stats_kernel(int32_t vocab, const void *__restrict__ logits,
                                                                int64_t row_stride, float *__restrict__ row_max,
                                                                float *__restrict__ row_sumexp, int64_t rows_first,
                                                                const void *__restrict__ logits_after) {
    constexpr int ELT = BF16 ? 2 : 4;
    constexpr int PER_VEC = 16 / ELT;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int64_t row = blockIdx.x;                      // rows beyond the first buffer's come from the second
    const char *row_ptr = row < rows_first
                              ? reinterpret_cast<const char *>(logits) + row * row_stride * ELT
                              : reinterpret_cast<const char *>(logits_after) + (row - rows_first) * row_stride * ELT;
    float m = -__builtin_inff(), s = 0.f;
    // a batch of values joins the running state with one rescale: max of the batch first, then its exponentials
    auto add_batch = [&](const float *x, int cnt) {
        float bm = -__builtin_inff();
        for (int j = 0; j < cnt; ++j) bm = fmaxf(bm, x[j]);
        if (bm == -__builtin_inff()) return;
        const float mm = fmaxf(m, bm);
        float add = 0.f;
        for (int j = 0; j < cnt; ++j) add += __expf(x[j] - mm);
        s = s * __expf(m - mm) + add;
        m = mm;
    };
    // scalar head up to the first 16-byte boundary, 16-byte body, scalar tail
    const uintptr_t addr = reinterpret_cast<uintptr_t>(row_ptr);
    int head = int(((16 - (addr & 15)) & 15) / ELT);
    if (head > vocab) head = vocab;
    const int nvec = (vocab - head) / PER_VEC;
    const int tail_start = head + nvec * PER_VEC;
    auto scalar_at = [&](int32_t i) -> float {
        if (BF16) return __uint_as_float(uint32_t(reinterpret_cast<const uint16_t *>(row_ptr)[i]) << 16);
        return reinterpret_cast<const float *>(row_ptr)[i];
    };
    // the elements before the first and behind the last 16-byte boundary are fetched ahead of the body and looked at after
    // it was issued: waited for at once they would cost a row two more round trips to memory
    const bool has_head = int(threadIdx.x) < head, has_tail = tail_start + int(threadIdx.x) < vocab;
    float head_x = 0.f, tail_x = 0.f;
    if (has_head) head_x = scalar_at(threadIdx.x);
    if (has_tail) tail_x = scalar_at(tail_start + threadIdx.x);
    bool head_due = has_head;
    const u32x4 *vec = reinterpret_cast<const u32x4 *>(row_ptr + size_t(head) * ELT);
    // kBatch loads are issued before the first of them is looked at (one load per lane in flight streams at the pace of
    // memory latency, not bandwidth); a slot past the end of the row reads the last chunk again and is ignored
    constexpr int kBatch = 8;
    for (int c0 = threadIdx.x; c0 < nvec; c0 += THREADS * kBatch) {
        u32x4 w[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) w[u] = __builtin_nontemporal_load(vec + min(c0 + u * THREADS, nvec - 1));
        if (head_due) add_batch(&head_x, 1);
        head_due = false;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (c0 + u * THREADS >= nvec) break;
            float x[PER_VEC];
            if (BF16) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[2 * j] = __uint_as_float(w[u][j] << 16);
                    x[2 * j + 1] = __uint_as_float(w[u][j] & 0xffff0000u);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = __uint_as_float(w[u][j]);
            }
            add_batch(x, PER_VEC);
        }
    }
    if (head_due) add_batch(&head_x, 1);                 // a row too short to give this lane a chunk
    if (has_tail) add_batch(&tail_x, 1);
    merge_state(m, s, lane_xor<32>(m), lane_xor<32>(s));
    merge_state(m, s, lane_xor<16>(m), lane_xor<16>(s));
    merge_state(m, s, lane_xor<8>(m), lane_xor<8>(s));
    merge_state(m, s, lane_xor<4>(m), lane_xor<4>(s));
    merge_state(m, s, lane_xor<2>(m), lane_xor<2>(s));
    merge_state(m, s, lane_xor<1>(m), lane_xor<1>(s));
    __shared__ float sm[THREADS / 64], ss[THREADS / 64];
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = m;
        ss[threadIdx.x >> 6] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float M = sm[0], S = ss[0];
        for (int w = 1; w < THREADS / 64; ++w) merge_state(M, S, sm[w], ss[w]);
        row_max[row] = M;
        row_sumexp[row] = S;
    }
}

hipError_t launch_softmax_stats(int64_t rows, int32_t vocab, int dtype, const void *logits, int64_t row_stride,
                                float *row_max, float *row_sumexp, hipStream_t stream, int64_t rows_after,
                                const void *logits_after) {
    const dim3 grid((unsigned)(rows + rows_after));
    if (dtype == GSD_BF16)
        hipLaunchKernelGGL((softmax_stats_kernel<256, true>), grid, dim3(256), 0, stream, vocab, logits, row_stride,
                           row_max, row_sumexp, rows, logits_after);
    else
        hipLaunchKernelGGL((softmax_stats_kernel<256, false>), grid, dim3(256), 0, stream, vocab, logits, row_stride,
                           row_max, row_sumexp, rows, logits_after);
    return hipGetLastError();
}

constexpr int kStochThreads = 1024;            // one per node in the first phase, one per vocabulary slice in the second

struct AcceptLds {
    int32_t L[GSD_MAX_NODES_PER_SEQ];
    int32_t path[GSD_MAX_NODES_PER_SEQ];
    int32_t back[GSD_MAX_NODES_PER_SEQ];
    uint32_t wave_best[kStochThreads / 64];
    int32_t grew[3];                   // of a round of the relaxation: some L has grown
    int32_t len, end;
};

// Writes accept_len, accept_path and end_node of the calling work-group's sequence.  Returns the end node (-1: the root)
// and, in `child`, whether one of the calling thread's nodes is a child of it.
template <int THREADS>
__device__ __forceinline__ int accept_phase(AcceptLds &s, const gsd_stochastic_desc &d, bool &child) {
    int32_t *L = s.L, *path_s = s.path, *back_s = s.back;
    uint32_t *wave_best = s.wave_best;
    static_assert(THREADS >= GSD_MAX_NODES_PER_SEQ && THREADS <= kStochThreads, "one thread per node");

    const int b = blockIdx.x;
    const int64_t base = d.node_offsets[b];
    int n = d.node_offsets[b + 1] - d.node_offsets[b];
    if (n > d.max_nodes) n = d.max_nodes;
    if (n < 0) n = 0;
    const float *root_max = d.row_max + d.total_nodes, *root_sum = d.row_sumexp + d.total_nodes;

    // One thread per node.  Whether an edge passes never changes, so every node tests its own parent edges once
    // (its coin against the LLM's probability of its token after that parent) and keeps the first four that pass
    // in registers; the loads of the four tests are issued together, with clamped indices instead of branches.
    constexpr int kRegParents = 4;
    const int i = threadIdx.x;
    const bool active = i < n;
    int par[kRegParents];          // parent id of a passing edge; -1 = root; -2 = no such edge, or it did not pass
#pragma unroll
    for (int x = 0; x < kRegParents; ++x) par[x] = -2;
    int32_t e_lo = 0, e_hi = 0;    // this node's slice of parent_idx
    int32_t r[kRegParents];        // its first entries as they stand there, the last one repeated
#pragma unroll
    for (int x = 0; x < kRegParents; ++x) r[x] = -2;
    int32_t tok = 0;
    bool tok_ok = false;           // a token outside the vocabulary is never accepted
    float coin = 0.f;              // accept_u * draft_prob: the edge passes iff coin < p_r(tok)
    // the LLM's probability of this node's token after parent r (a well-formed parent, -1 = the root)
    auto prob_after = [&](int r) -> float {
        const void *rows = r == -1 ? d.root_logits : d.logits;
        const int64_t row = r == -1 ? int64_t(b) : base + r;
        const float mx = r == -1 ? root_max[b] : d.row_max[base + r];
        const float sm = r == -1 ? root_sum[b] : d.row_sumexp[base + r];
        return __expf(load_logit(rows, row * d.row_stride + tok, d.dtype) - mx) / sm;
    };
    if (active) {
        e_lo = d.parent_offsets[base + i];
        e_hi = d.parent_offsets[base + i + 1];
        tok = d.tokens[base + i];
        coin = d.accept_u[base + i] * d.draft_prob[base + i];
        tok_ok = tok >= 0 && tok < d.vocab;
        if (!tok_ok) tok = 0;                                  // keeps the gathers below in bounds
        if (e_hi > e_lo) {
#pragma unroll
            for (int x = 0; x < kRegParents; ++x) r[x] = d.parent_idx[min(e_lo + x, e_hi - 1)];
#pragma unroll
            for (int x = 0; x < kRegParents; ++x) {
                const bool wf = e_lo + x < e_hi && r[x] >= -1 && r[x] < i;
                const float pr = prob_after(wf ? r[x] : -1);
                if (wf && tok_ok && coin < pr) par[x] = r[x];
            }
        }
        L[i] = -1;
    }
    if (i < 3) s.grew[i] = 0;
    const bool more = active && e_hi - e_lo > kRegParents;     // rare: a node with more than four parents
    auto passes = [&](int r) -> bool { return r >= -1 && r < i && tok_ok && coin < prob_after(r); };
    __syncthreads();

    // L[i] = 1 + max L[parent] by relaxation.  Values only grow and whatever is read is the length of a path that exists, so the
    // waves follow their own nodes for a few steps and then meet to find out whether all have come to rest (256 nodes: 1.35 us,
    // 2.3 when every step was a sweep with a barrier and a reduction).
    // Further parents are tested anew in every step: a wave that has some takes one step at a time.
    const int steps = __any(more) ? 1 : 4;
    int32_t mine = -1;             // L[i]
    for (int round = 0; round <= n; ++round) {
        bool grew = false;
        if (active) {
#pragma unroll 1
            for (int step = 0; step < steps; ++step) {
                int32_t best = mine;
#pragma unroll
                for (int x = 0; x < kRegParents; ++x) {
                    const int32_t l = __hip_atomic_load(&L[par[x] >= 0 ? par[x] : i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const int32_t lr = par[x] >= 0 ? l : (par[x] == -1 ? 0 : -1);
                    if (lr >= 0 && lr + 1 > best) best = lr + 1;
                }
                if (more) {
                    for (int e = e_lo + kRegParents; e < e_hi; ++e) {
                        const int r = d.parent_idx[e];
                        if (!passes(r)) continue;
                        const int32_t lr = r == -1 ? 0 : __hip_atomic_load(&L[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (lr >= 0 && lr + 1 > best) best = lr + 1;
                    }
                }
                const bool up = best != mine;
                if (up) {
                    mine = best;
                    grew = true;
                    __hip_atomic_store(&L[i], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                if (!__any(up)) break;
            }
        }
        // three flags in turn: one is written, one read, and the one that everybody has read is cleared
        const int at = round % 3;
        if (grew) s.grew[at] = 1;
        __syncthreads();
        if (i == 0) s.grew[(round + 2) % 3] = 0;
        if (s.grew[at] == 0) break;
    }

    // back pointer of every accepted node: the smallest-id passing parent that ends a path one node shorter
    if (active && mine > 0) {
        int32_t chosen = 0x7fffffff;
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) {
            const int32_t l = L[par[x] >= 0 ? par[x] : i];
            const int32_t lr = par[x] >= 0 ? l : (par[x] == -1 ? 0 : -1);
            if (lr == mine - 1 && par[x] < chosen) chosen = par[x];
        }
        if (more) {
            for (int e = e_lo + kRegParents; e < e_hi; ++e) {
                const int r = d.parent_idx[e];
                if (!passes(r)) continue;
                const int32_t lr = (r == -1) ? 0 : L[r];
                if (lr == mine - 1 && r < chosen) chosen = r;
            }
        }
        back_s[i] = chosen;
    }

    uint32_t key = 0;                                    // largest L, then smallest id
    if (active && mine > 0) key = uint32_t(mine) * 1024u + uint32_t(1023 - i);
    key = max(key, lane_xor<32>(key));
    key = max(key, lane_xor<16>(key));
    key = max(key, lane_xor<8>(key));
    key = max(key, lane_xor<4>(key));
    key = max(key, lane_xor<2>(key));
    key = max(key, lane_xor<1>(key));
    if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t k = 0;
        for (int w = 0; w < THREADS / 64; ++w) k = wave_best[w] > k ? wave_best[w] : k;
        const int32_t len = int32_t(k / 1024u);
        int32_t v = (len > 0) ? int32_t(1023u - (k % 1024u)) : -1;
        s.len = len;
        s.end = v;
        d.accept_len[b] = len;
        d.end_node[b] = v;
        for (int pos = len - 1; pos >= 0 && v >= 0 && v < n; --pos) {   // L drops by one per step: the root's child sits at pos 0
            path_s[pos] = v;
            v = back_s[v];
        }
    }
    __syncthreads();
    const int32_t len = s.len, end = s.end;
    int32_t *out = d.accept_path + int64_t(b) * d.max_nodes;
    for (int x = threadIdx.x; x < d.max_nodes; x += THREADS) out[x] = (x < len) ? path_s[x] : -1;
    child = false;
    if (active && e_hi > e_lo) {
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) child |= r[x] == end;
        for (int e = e_lo + kRegParents; e < e_hi; ++e) child |= d.parent_idx[e] == end;
    }
    return end;
}

constexpr int kResampleThreads = kStochThreads;
constexpr int kResampleWaves = kResampleThreads / 64;

__device__ __forceinline__ void merge_lanes(float &m, float &s) {      // of a wave, in every lane
    merge_state(m, s, lane_xor<32>(m), lane_xor<32>(s));
    merge_state(m, s, lane_xor<16>(m), lane_xor<16>(s));
    merge_state(m, s, lane_xor<8>(m), lane_xor<8>(s));
    merge_state(m, s, lane_xor<4>(m), lane_xor<4>(s));
    merge_state(m, s, lane_xor<2>(m), lane_xor<2>(s));
    merge_state(m, s, lane_xor<1>(m), lane_xor<1>(s));
}

// The states of the work-group's 16 waves merged in their order, by one wave, a state per lane: the running maxima and both
// factors of every merge at once, which leaves one multiply-add per state in the chain.
__device__ __forceinline__ void merge_waves(const float *red_m, const float *red_s, float &m, float &s) {
    static_assert(kResampleWaves == 16, "a row of 16 lanes");
    const int w = threadIdx.x & 15;
    const float empty = -__builtin_inff(), mw = red_m[w];
    auto from_below = [&](float x, auto shift) -> float {              // lane w - shift of the row; none: empty
        constexpr int kRowShr = 0x110;
        return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(empty), __float_as_uint(x), kRowShr + decltype(shift)::value,
                                                           0xf, 0xf, false));
    };
    float top = mw;
    top = fmaxf(top, from_below(top, std::integral_constant<int, 1>{}));
    top = fmaxf(top, from_below(top, std::integral_constant<int, 2>{}));
    top = fmaxf(top, from_below(top, std::integral_constant<int, 4>{}));
    top = fmaxf(top, from_below(top, std::integral_constant<int, 8>{}));
    const float below = from_below(top, std::integral_constant<int, 1>{});
    const bool none = top == empty;                                    // all states up to this one are empty
    const uint32_t keep = __float_as_uint(none ? 0.f : __expf(below - top));
    const uint32_t add = __float_as_uint(red_s[w] * (none ? 0.f : __expf(mw - top)));
    s = red_s[0];
#pragma unroll
    for (int x = 1; x < kResampleWaves; ++x)
        s = __builtin_fmaf(s, __uint_as_float(__builtin_amdgcn_readlane(keep, x)), __uint_as_float(__builtin_amdgcn_readlane(add, x)));
    m = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(top), 15));
}

// x / d, correctly rounded, for many x and one d from [1, 2^31): two corrections of x * (1/d).  The first leaves a quotient
// within an ulp, from which, with a correctly rounded reciprocal, the second rounds correctly (Markstein 1990); remainders are
// exact and quotients normal down to x = 2^-94, below which it is left to the compiler's division (5 instructions instead of 11 and a
// reciprocal each).
struct Divisor {
    float d, inverse;
    __device__ __forceinline__ explicit Divisor(float by) : d(by), inverse(1.f / by) {}
    __device__ __forceinline__ float operator()(float x) const {
        float q = x * inverse;
        q = __builtin_fmaf(__builtin_fmaf(-q, d, x), inverse, q);
        q = __builtin_fmaf(__builtin_fmaf(-q, d, x), inverse, q);
        if (__builtin_expect(__any(__float_as_uint(x) - 1u < __float_as_uint(0x1p-94f) - 1u), 0)) q = x / d;
        return q;
    }
};

// The draw for any vocabulary, type and alignment.  A thread's slice is contiguous in memory, so lanes that fetched their
// own slices one element after the other would touch 64 lines with every load; instead neighbouring lanes fetch
// neighbouring elements, all slices a segment of SEG_BYTES at a time, into LDS, where a slice starts an odd number of
// words after the one before it (no bank conflicts when every lane then reads its own).  The slice that holds the target
// is weighed by the whole work-group and walked by one thread.  Bound by the chain of these phases on one CU.
// 8 sequences of 128 nodes, whole call: 32003 bf16 tokens 66.4 -> 43.7 us; 4 sequences, 64000 tokens: 108 -> 61.7;
// 2 sequences, 64001 fp32 tokens: 98.5 -> 62.7, against a kernel that fetched slices lane by lane.  With the scan and the
// divisions below: 8 of 64 nodes, 32003 tokens 34.4 -> 31.6, 4 of 64, 64000 tokens 53.4 -> 48.3.
template <bool BF16, int SEG_BYTES>
__device__ __forceinline__ void resample_phase(const gsd_stochastic_desc &d, int end, bool child) {
    constexpr int ELT = BF16 ? 2 : 4;
    constexpr int kSeg = SEG_BYTES / ELT;                         // elements of a slice that are in LDS at a time
    constexpr int kStride = SEG_BYTES / 4 + 1;                    // words from one slice's segment to the next
    constexpr int kWaves = kResampleWaves;
    __shared__ uint32_t seg_p[kResampleThreads * kStride], seg_q[kResampleThreads * kStride];
    constexpr int kBefore = kResampleThreads - 64;                // zeros in front: what the first waves find before themselves
    __shared__ float part[kResampleThreads], part_of_waves[kBefore + kResampleThreads];
    __shared__ float red_m[kWaves], red_s[kWaves], stat[2];
    __shared__ int owner_s, pick_s;

    const int t = threadIdx.x;
    const int b = blockIdx.x;
    const int64_t base = d.node_offsets[b];
    const int V = d.vocab;
    if (t == 0) {
        owner_s = 0x7fffffff;
        pick_s = -1;
    }
    if (t < kBefore) part_of_waves[t] = 0.f;
    const int64_t row_off = (end < 0 ? int64_t(b) : base + end) * d.row_stride;
    const char *p_row = reinterpret_cast<const char *>(end < 0 ? d.root_logits : d.logits) + row_off * ELT;
    const char *q_row = reinterpret_cast<const char *>(end < 0 ? d.root_draft_logits : d.draft_logits) + row_off * ELT;
    const float p_max = end < 0 ? d.row_max[d.total_nodes + b] : d.row_max[base + end];
    const float p_sum = end < 0 ? d.row_sumexp[d.total_nodes + b] : d.row_sumexp[base + end];
    auto raw = [&](const char *row, int x) -> uint32_t {
        if (BF16) return reinterpret_cast<const uint16_t *>(row)[x];
        return reinterpret_cast<const uint32_t *>(row)[x];
    };
    auto value = [&](uint32_t v) -> float { return __uint_as_float(BF16 ? v << 16 : v); };

    // the draft row's own (max, sum)
    float m = -__builtin_inff(), s = 0.f;
    constexpr int kBatch = 16;
    for (int x0 = t; x0 < V; x0 += kResampleThreads * kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (x0 - t + u * kResampleThreads >= V) break;        // uniform
            v[u] = raw(q_row, min(x0 + u * kResampleThreads, V - 1));
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (x0 + u * kResampleThreads >= V) break;
            const float x = value(v[u]);
            if (fabsf(x) < __builtin_inff()) {                    // merge_state(m, s, x, 1) with the one exponential that
                const float e = __expf(x > m ? m - x : x - m);    // is not exp(0)
                s = x > m ? fmaf(s, e, 1.f) : s + e;
                m = fmaxf(m, x);
            } else {
                merge_state(m, s, x, 1.f);
            }
        }
    }
    merge_lanes(m, s);
    if ((t & 63) == 0) {
        red_m[t >> 6] = m;
        red_s[t >> 6] = s;
    }
    const bool use_residual = __syncthreads_or(child) != 0;       // does the end node (or the root) have children ?
    if (t < 64) {
        float M, S;
        merge_waves(red_m, red_s, M, S);
        if (t == 0) {
            stat[0] = M;
            stat[1] = S;
        }
    }
    __syncthreads();
    const float q_max = stat[0];
    const Divisor by_p(p_sum), by_q(stat[1]);
    auto weight = [&](uint32_t vp, uint32_t vq, bool residual) -> float {
        const float p = by_p(__expf(value(vp) - p_max));
        if (!residual) return p;
        const float q = by_q(__expf(value(vq) - q_max));
        return fmaxf(p - q, 0.f);
    };

    const int per = (V + kResampleThreads - 1) / kResampleThreads;
    const int x0 = t * per;
    // weight of this thread's slice, in ascending token order
    auto slice_sum = [&](bool residual) -> float {
        float local = 0.f;
        for (int g0 = 0; g0 < per; g0 += kSeg) {
            const int width = min(kSeg, per - g0);                // elements per slice in this turn
            int lg = 0;                                           // 2^lg >= width lanes fetch a slice's segment
            while ((1 << lg) < width) ++lg;
            const int e = t & ((1 << lg) - 1), first = t >> lg, step = kResampleThreads >> lg, rounds = 1 << lg;
            __syncthreads();                                      // the segment before this one has been read
            constexpr int kFetch = 8;
            for (int r0 = 0; r0 < rounds; r0 += kFetch) {
                uint32_t vp[kFetch], vq[kFetch];
#pragma unroll
                for (int u = 0; u < kFetch; ++u) {
                    if (r0 + u >= rounds) break;                  // uniform
                    const int slice = first + (r0 + u) * step;
                    const int x = min(slice * per + g0 + e, V - 1);
                    vp[u] = raw(p_row, x);
                    vq[u] = raw(q_row, x);
                }
#pragma unroll
                for (int u = 0; u < kFetch; ++u) {
                    const int slice = first + (r0 + u) * step;
                    if (r0 + u >= rounds) break;
                    if (e < width) {
                        if (BF16) {
                            reinterpret_cast<uint16_t *>(seg_p)[slice * 2 * kStride + e] = uint16_t(vp[u]);
                            reinterpret_cast<uint16_t *>(seg_q)[slice * 2 * kStride + e] = uint16_t(vq[u]);
                        } else {
                            seg_p[slice * kStride + e] = vp[u];
                            seg_q[slice * kStride + e] = vq[u];
                        }
                    }
                }
            }
            __syncthreads();
            constexpr int kPerWord = 4 / ELT;
#pragma unroll 4
            for (int w = 0; w < SEG_BYTES / 4; ++w) {
                if (w * kPerWord >= width) break;                 // uniform
                const uint32_t wp = seg_p[t * kStride + w], wq = seg_q[t * kStride + w];
#pragma unroll
                for (int h = 0; h < kPerWord; ++h) {
                    const int i = g0 + w * kPerWord + h;
                    const uint32_t vp = BF16 ? (h ? wp >> 16 : wp & 0xffffu) : wp;
                    const uint32_t vq = BF16 ? (h ? wq >> 16 : wq & 0xffffu) : wq;
                    if (i < per && x0 + i < V) local += weight(vp, vq, residual);
                }
            }
        }
        return local;
    };
    // Inclusive scan of the slices' weights in one fixed order, that of ten doubling steps: value t takes in value t - 1, then
    // t - 2, t - 4, ... t - 512, each as the step before left it.  The steps up to 32 reach into the wave before at most, so a
    // wave takes them on its own, with that wave's values in a second register; the others stay in the lane, sixteen
    // values from LDS.  Three barriers instead of eleven, 2.9 instead of 5.4 us.  A wave with fewer than sixteen before it finds
    // zeros there; deciding that per value keeps sixteen lane masks, which spills scalar registers where two work-groups share a
    // CU (512 sequences of 4 nodes, 1000 tokens, whole call 19.8 us instead of 19.4; 2048 of 2 nodes 49.5 instead of 47.2).
    float before = 0.f, upto = 0.f, total = 0.f;
    const int lane = t & 63, wave = t >> 6;
    auto scan = [&](bool residual) {
        float a = slice_sum(residual);
        part[t] = a;
        __syncthreads();
        float prev = wave > 0 ? part[t - 64] : 0.f;              // (lanes below a step's reach are not needed after it)
#pragma unroll
        for (int dd = 1; dd < 64; dd <<= 1) {
            const int src = (lane - dd) & 63;
            const float from_a = __shfl(a, src, 64), from_prev = __shfl(prev, src, 64);
            if (t >= dd) a += lane >= dd ? from_a : from_prev;
            prev += lane >= dd ? from_prev : 0.f;
        }
        part_of_waves[kBefore + t] = a;
        __syncthreads();
        float x[kWaves];
#pragma unroll
        for (int j = 0; j < kWaves; ++j) x[j] = part_of_waves[kBefore + t - 64 * j];
#pragma unroll
        for (int step = 1; step < kWaves; step <<= 1)            // x[j] stands for wave - j
#pragma unroll
            for (int j = 0; j + step < kWaves; j += 2 * step) x[j] += x[j + step];
        upto = x[0];
        part[t] = upto;
        __syncthreads();
        before = t > 0 ? part[t - 1] : 0.f;
        total = part[kResampleThreads - 1];
    };
    bool residual = use_residual;
    scan(residual);
    if (residual && !(total > 0.f)) {                             // empty residual: draw from p
        __syncthreads();
        residual = false;
        scan(false);
    }
    const float target = d.resample_u[b] * total;
    // the owner of the target: the smallest token whose cumulative weight exceeds the target is in its slice
    const bool mine = before <= target && target < upto;
    if (mine) atomicMin(&owner_s, t);
    __syncthreads();
    const int owner = owner_s;
    if (owner < kResampleThreads) {                               // uniform
        float run = before;
        int pick = -1, last = -1;
        float *weights = reinterpret_cast<float *>(seg_p);
        for (int c0 = 0; c0 < per; c0 += kResampleThreads) {
            const int i = c0 + t, x = owner * per + i;
            const bool in = i < per && x < V;
            if (in) weights[t] = weight(raw(p_row, x), raw(q_row, x), residual);
            __syncthreads();
            if (t == owner) {
                const int count = min(min(per - c0, kResampleThreads), V - (x0 + c0));
#pragma unroll 8
                for (int k = 0; k < count; ++k) {
                    const float w = weights[k];
                    run += w;
                    if (w > 0.f) last = x0 + c0 + k;
                    if (pick < 0 && run > target) pick = x0 + c0 + k;
                }
            }
            __syncthreads();
        }
        if (t == owner) pick_s = pick >= 0 ? pick : last;         // rounding inside the slice: its last token with weight
    }
    __syncthreads();
    if (pick_s < 0) {                                             // target == total by rounding: the last token with weight
        int last = -1;
        for (int x = t; x < V; x += kResampleThreads)
            if (weight(raw(p_row, x), raw(q_row, x), residual) > 0.f) last = x;
        for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off, 64));
        if ((t & 63) == 0) red_m[t >> 6] = __int_as_float(last);
        __syncthreads();
        if (t == 0) {
            int best = 0;
            for (int w = 0; w < kWaves; ++w) best = max(best, __float_as_int(red_m[w]));
            pick_s = best;
        }
    }
    if (t == 0) d.bonus_token[b] = pick_s;
}

// The same draw for rows whose per-thread slice fits registers (the launcher checks: the slice is a whole number of
// 16-byte runs, at most kHeld values, rows start on 16-byte boundaries, the vocabulary ends on one): a thread fetches
// its slice of both rows once, all loads in flight together, and every later step works from those registers: the
// draft row's normaliser, the slice's weight sum, and (for the one thread that owns the target) the walk.  Scans go
// through wave shuffles and one LDS hop instead of a log-step LDS scan; the order of every sum is fixed.
constexpr int kHeld = 32;

template <bool BF16>
__device__ __forceinline__ void resample_held_phase(const gsd_stochastic_desc &d, int end, bool child) {
    constexpr int ELT = BF16 ? 2 : 4;
    constexpr int PER_VEC = 16 / ELT;
    constexpr int KV = kHeld / PER_VEC;
    constexpr int kWaves = kResampleWaves;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __shared__ float red_m[kWaves], red_s[kWaves], stat[2], wave_sum[2][kWaves];
    __shared__ int pick_s;

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int b = blockIdx.x;
    const int64_t base = d.node_offsets[b];
    const int V = d.vocab;
    if (t == 0) pick_s = -1;

    const int64_t row_off = (end < 0 ? int64_t(b) : base + end) * d.row_stride;
    const char *p_ptr = reinterpret_cast<const char *>(end < 0 ? d.root_logits : d.logits) + row_off * ELT;
    const char *q_ptr = reinterpret_cast<const char *>(end < 0 ? d.root_draft_logits : d.draft_logits) + row_off * ELT;
    const int per = (V + kResampleThreads - 1) / kResampleThreads;
    const int x0 = t * per;
    const int nvec = x0 < V ? min(per, V - x0) / PER_VEC : 0;     // whole 16-byte runs: the vocabulary ends on one
    u32x4 raw_p[KV], raw_q[KV];
#pragma unroll
    for (int j = 0; j < KV; ++j) {                                // a run this thread does not have reads the row's first
        const int64_t off = (j < nvec ? int64_t(x0) + j * PER_VEC : 0) * ELT;
        raw_q[j] = *reinterpret_cast<const u32x4 *>(q_ptr + off);
        raw_p[j] = *reinterpret_cast<const u32x4 *>(p_ptr + off);
    }
    const float p_max = end < 0 ? d.row_max[d.total_nodes + b] : d.row_max[base + end];
    const float p_sum = end < 0 ? d.row_sumexp[d.total_nodes + b] : d.row_sumexp[base + end];

    auto value = [&](const u32x4 v, int e) -> float {
        if (BF16) return (e & 1) ? __uint_as_float(v[e >> 1] & 0xffff0000u) : __uint_as_float(v[e >> 1] << 16);
        return __uint_as_float(v[e]);
    };
    // the draft row's own (max, sum)
    float m = -__builtin_inff(), sum = 0.f;
#pragma unroll
    for (int j = 0; j < KV; ++j)
        if (j < nvec) {
#pragma unroll
            for (int e = 0; e < PER_VEC; ++e) m = fmaxf(m, value(raw_q[j], e));
        }
    if (m > -__builtin_inff()) {
#pragma unroll
        for (int j = 0; j < KV; ++j)
            if (j < nvec) {
#pragma unroll
                for (int e = 0; e < PER_VEC; ++e) sum += __expf(value(raw_q[j], e) - m);
            }
    }
    merge_lanes(m, sum);
    if (lane == 0) {
        red_m[wave] = m;
        red_s[wave] = sum;
    }
    const bool use_residual = __syncthreads_or(child) != 0;       // does the end node (or the root) have children ?
    if (wave == 0) {
        float M, S;
        merge_waves(red_m, red_s, M, S);
        if (lane == 0) {
            stat[0] = M;
            stat[1] = S;
        }
    }
    __syncthreads();
    const float q_max = stat[0], q_sum = stat[1];

    const float p_scale = 1.f / p_sum, q_scale = 1.f / q_sum;     // one division per row instead of one per token
    auto weight_of = [&](float lp, float lq, bool residual) -> float {
        const float pp = __expf(lp - p_max) * p_scale;
        return residual ? fmaxf(pp - __expf(lq - q_max) * q_scale, 0.f) : pp;
    };
    // the cumulative weight before this thread's slice and up to its end: the slice in ascending token order, the
    // wave in lane order, the waves in their order
    float before = 0.f, upto = 0.f, total = 0.f;
    float held[kHeld];                                            // the slice's weights: the owner walks them
    auto scan = [&](bool residual, int turn) {
        float local = 0.f;
#pragma unroll
        for (int j = 0; j < KV; ++j)
#pragma unroll
            for (int e = 0; e < PER_VEC; ++e) {
                float &w = held[j * PER_VEC + e];
                w = 0.f;
                if (j < nvec) w = weight_of(value(raw_p[j], e), value(raw_q[j], e), residual);
                local += w;
            }
        float incl = local;
#pragma unroll
        for (int dd = 1; dd < 64; dd <<= 1) {
            const float up = __shfl_up(incl, dd, 64);
            if (lane >= dd) incl += up;
        }
        const float left = __shfl_up(incl, 1, 64);
        if (lane == 63) wave_sum[turn][wave] = incl;
        __syncthreads();
        float run = 0.f, mine_base = 0.f;
        for (int w = 0; w < kWaves; ++w) {
            if (w == wave) mine_base = run;
            run += wave_sum[turn][w];
        }
        total = run;
        before = lane == 0 ? mine_base : mine_base + left;
        upto = mine_base + incl;
    };
    bool residual = use_residual;
    scan(residual, 0);
    if (residual && !(total > 0.f)) {                        // empty residual: draw from p
        residual = false;
        scan(false, 1);
    }
    const float target = d.resample_u[b] * total;
    // the owner of the target walks its slice; the smallest token whose cumulative weight exceeds the target
    if (before <= target && target < upto) {
        float run = before;
        int pick = -1, last = -1;
#pragma unroll
        for (int j = 0; j < KV; ++j)
            if (j < nvec) {
#pragma unroll
                for (int e = 0; e < PER_VEC; ++e) {
                    const float w = held[j * PER_VEC + e];
                    run += w;
                    if (w > 0.f) last = x0 + j * PER_VEC + e;
                    if (pick < 0 && run > target) pick = x0 + j * PER_VEC + e;
                }
            }
        pick_s = pick >= 0 ? pick : last;                   // rounding inside the slice: its last token with weight
    }
    __syncthreads();
    if (pick_s < 0) {                                       // target == total by rounding: the last token with weight
        int last = -1;
#pragma unroll
        for (int j = 0; j < KV; ++j)
            if (j < nvec) {
#pragma unroll
                for (int e = 0; e < PER_VEC; ++e)
                    if (held[j * PER_VEC + e] > 0.f) last = x0 + j * PER_VEC + e;
            }
        for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off, 64));
        __shared__ int wave_last[kWaves];
        if (lane == 0) wave_last[wave] = last;
        __syncthreads();
        if (t == 0) {
            int best = 0;
            for (int w = 0; w < kWaves; ++w) best = max(best, wave_last[w]);
            pick_s = best;
        }
        __syncthreads();
    }
    if (t == 0) d.bonus_token[b] = pick_s;
}

enum class Resample { general_f32, general_bf16, held_f32, held_bf16 };

// `child`: whether one of the calling thread's nodes, or edges, has the end node as a parent
template <Resample KIND, int SEG_BYTES>
__device__ __forceinline__ void draw(const gsd_stochastic_desc &d, int end, bool child) {
    if constexpr (KIND == Resample::general_f32 || KIND == Resample::general_bf16)
        resample_phase<KIND == Resample::general_bf16, SEG_BYTES>(d, end, child);
    else
        resample_held_phase<KIND == Resample::held_bf16>(d, end, child);
}

template <Resample KIND>
__global__ __launch_bounds__(kStochThreads) void accept_and_resample_kernel(const gsd_stochastic_desc d) {
    __shared__ AcceptLds s;
    bool child = false;
    const int end = __builtin_amdgcn_readfirstlane(accept_phase<kStochThreads>(s, d, child));
    draw<KIND, 64>(d, end, child);
}

// The phases one by one, for more sequences than the chip has CUs: a CU then takes as many work-groups at a time as each
// phase leaves room for (4, and 1 or 2) instead of one.
constexpr int kAcceptOnlyThreads = 512;
__global__ __launch_bounds__(kAcceptOnlyThreads) void accept_stochastic_kernel(const gsd_stochastic_desc d) {
    __shared__ AcceptLds s;
    bool child = false;
    accept_phase<kAcceptOnlyThreads>(s, d, child);
}

// (The general draw has to leave room for a second work-group: at 7 wavefronts to a SIMD 512 sequences over 1000 tokens take
// 22.8 us a call instead of 19.5.)
template <Resample KIND>
__global__ __launch_bounds__(kResampleThreads, KIND == Resample::general_f32 || KIND == Resample::general_bf16 ? 8 : 4)
void resample_kernel(const gsd_stochastic_desc d) {
    const int64_t base = d.node_offsets[blockIdx.x];
    const int n = max(0, min(d.node_offsets[blockIdx.x + 1] - int32_t(base), d.max_nodes));
    const int end = __builtin_amdgcn_readfirstlane(d.end_node[blockIdx.x]);
    bool child = false;
    const int32_t e1 = d.parent_offsets[base + n];
    for (int e = d.parent_offsets[base] + int32_t(threadIdx.x); e < e1; e += kResampleThreads) child |= d.parent_idx[e] == end;
    draw<KIND, 16>(d, end, child);
}

hipError_t launch_accept_stochastic(const gsd_stochastic_desc &d, hipStream_t stream) {
    // the node rows and, behind them, the root rows: one launch
    hipError_t err = launch_softmax_stats(d.total_nodes, d.vocab, d.dtype, d.logits, d.row_stride, d.row_max,
                                          d.row_sumexp, stream, d.batch, d.root_logits);
    if (err != hipSuccess) return err;
    // slices that fit registers: see resample_held_phase
    const int elt = d.dtype == GSD_BF16 ? 2 : 4;
    const int per = (d.vocab + kResampleThreads - 1) / kResampleThreads;
    auto aligned = [&](const void *ptr) { return reinterpret_cast<uintptr_t>(ptr) % 16 == 0; };
    const bool held = per <= kHeld && (per * elt) % 16 == 0 && (int64_t(d.vocab) * elt) % 16 == 0 &&
                      (d.row_stride * elt) % 16 == 0 && aligned(d.logits) && aligned(d.root_logits) &&
                      aligned(d.draft_logits) && aligned(d.root_draft_logits);
    // One launch while every sequence has a CU for itself, two beyond: 8 sequences of 256 nodes, 32000 tokens, 16.7 us against
    // 7.0 + 11.7; whole calls of 512 of 4 nodes, 100 tokens, 23.7 us in one and 18.8 in two, 4096 of 1 node, 500 tokens, 142 and 78.
    constexpr int kCus = 256;
    const dim3 grid(d.batch), block(kStochThreads);
    if (d.batch > kCus) {
        hipLaunchKernelGGL(accept_stochastic_kernel, grid, dim3(kAcceptOnlyThreads), 0, stream, d);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
#define GSD_DRAW(KIND)                                                                                               \
    do {                                                                                                            \
        if (d.batch > kCus) hipLaunchKernelGGL(resample_kernel<KIND>, grid, block, 0, stream, d);                     \
        else hipLaunchKernelGGL(accept_and_resample_kernel<KIND>, grid, block, 0, stream, d);                        \
    } while (0)
    if (held && d.dtype == GSD_BF16) GSD_DRAW(Resample::held_bf16);
    else if (held) GSD_DRAW(Resample::held_f32);
    else if (d.dtype == GSD_BF16) GSD_DRAW(Resample::general_bf16);
    else GSD_DRAW(Resample::general_f32);
#undef GSD_DRAW
    return hipGetLastError();
}

}  // namespace gsd
