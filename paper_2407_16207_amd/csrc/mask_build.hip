// Visibility-mask builder: ancestor closure of the token graph, one work-group per sequence.
//
// Paper Section 4.1 lets a flattened token attend only to its ancestors; on the merged graph of Section 5.3
// that set is the closure over all parent edges,
//     row[i] = bit(i) | OR_{p in parents(i)} row[p].
// Parents come before their children, so the matrix of rows is lower triangular; it is built in blocks of 64 x 64 bits, one
// wavefront per column of blocks and one lane per row:
//   the block on the diagonal   the closure of the edges that stay within 64 nodes, by Warshall's algorithm: node k's row is
//                               final when it is its turn, and goes to every lane that has bit k (readlane, two or three
//                               vector instructions for each of 64 steps);
//   a block below it            what the parents outside the block's own 64 rows have in this column (read from LDS: a few
//                               words per lane), spread over the rows by the diagonal block: row i takes it from every node j
//                               that it descends from within its 64, handed out by readlane, nodes without such parents left out.
// A wavefront needs the diagonal blocks of the others, and otherwise only words of its own column: one barrier in all, however
// deep the graph.  Bound by latency: three round trips to memory (offsets, parent lists) and 0.5 us for the diagonal;
// following the layers of the graph instead, one after the other with a flag per node, took 0.2 us for each of them.
// Launches in a replayed graph, against that (us): 64 nodes in 8 layers 3.9 -> 2.9, 8 x 256 in 32 layers 9.3 -> 4.9, 32 x 512 in
// 64 layers 19.3 -> 7.5; random graphs 77 nodes 3.5-5.1 -> 3.9, 8 x 512 15.6-19.9 -> 12.9; a chain of 512 101 -> 7.1.
// Shallow graphs have little for it to save.  Blocks without edges within (children of the root, layers of 64 and more) skip both
// kinds of steps, which costs the others less than 1 %: a star of 77 nodes 3.5 -> 3.0 (2.9 by layers), 2 layers of 64 4.4 -> 2.9
// (3.0), 2 of 256 9.9 -> 5.6 (15.0).  Behind following the layers are still 4 layers of 32, 3.9 (3.4), 5 of 25, 4.1 (3.6), and random
// trees of 128 to 256 nodes, by up to a tenth; leaving out eight nodes at a time by whether they have children in the block mends a third of
// that at most and takes every deep graph 3-6 % more.
#include "gsd_internal.h"

namespace gsd {

constexpr int kEdgeCacheInts = 6144;   // parent lists with more than four entries somewhere are staged in LDS when they fit

// W: words per row that are computed = wavefronts
template <int W>
__global__ __launch_bounds__(64 * W) void build_mask_kernel(
    int32_t max_nodes, int32_t words_per_row, const int32_t *__restrict__ node_offsets,
    const int32_t *__restrict__ parent_offsets, const int32_t *__restrict__ parent_idx, uint64_t *__restrict__ mask,
    int32_t *__restrict__ dag_error_flag) {
    constexpr int kNodes = 64 * W;
    constexpr uint32_t kNone = 0xffff;                       // no parent in an earlier block of rows
    __shared__ uint64_t diagonal[kNodes];                    // word i / 64 of row i
    __shared__ uint64_t outer[kNodes];                       // a node's first four parents in earlier blocks, 16 bits each
    __shared__ uint64_t column[W][kNodes + 1];               // word w of the rows, by wavefront w; the last one stays 0
    __shared__ int32_t offset[kNodes + 1];
    __shared__ int32_t wave_says[W];                         // bit 0: some node has more than four parents; 1: edges within the block
    __shared__ int32_t edge_cache[kEdgeCacheInts];

    const int b = blockIdx.x;
    const int64_t base = node_offsets[b];
    int n = node_offsets[b + 1] - node_offsets[b];
    bool bad = false;
    if (n > max_nodes) {                                     // caller's bound was wrong: flag, process what fits
        n = max_nodes;
        bad = true;
    }
    if (n <= 0) return;

    const int i = threadIdx.x, lane = i & 63, w = __builtin_amdgcn_readfirstlane(i >> 6);
    constexpr int kRegParents = 4;
    int e_lo = 0, e_hi = 0;
    if (i < n) {
        e_lo = parent_offsets[base + i];
        e_hi = parent_offsets[base + i + 1];
        offset[i] = e_lo;
        if (i == n - 1) offset[n] = e_hi;
    }
    const bool more = e_hi - e_lo > kRegParents;             // rare: a node with more than four parents
    uint64_t own = i < n ? uint64_t(1) << lane : 0;
    {
        int par[kRegParents];
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) par[x] = -1;
        if (e_hi > e_lo) {
#pragma unroll
            for (int x = 0; x < kRegParents; ++x) par[x] = parent_idx[min(e_lo + x, e_hi - 1)];
        }
        uint64_t packed = 0;
        auto take = [&](int p) {
            if (p >= 0 && p < i) {
                if (p >> 6 == w) own |= uint64_t(1) << (p & 63);
            } else if (p != -1) {
                bad = true;
            }
        };
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) {
            const int p = e_lo + x < e_hi ? par[x] : -1;
            take(p);
            packed |= uint64_t(p >= 0 && p < 64 * w ? uint32_t(p) : kNone) << (16 * x);
        }
        outer[i] = packed;
        constexpr int kBatch = 8;
        for (int e0 = e_lo + kRegParents; e0 < e_hi; e0 += kBatch) {
            int p[kBatch];
#pragma unroll
            for (int x = 0; x < kBatch; ++x) p[x] = parent_idx[min(e0 + x, e_hi - 1)];
#pragma unroll
            for (int x = 0; x < kBatch; ++x)
                if (e0 + x < e_hi) take(p[x]);
        }
    }

    // The diagonal block.  Step k hands the row of lane k to the lanes that have bit k; rows of the lower half have no bits in
    // the upper.  (One block alone: nearly all such graphs have edges, and a branch that waits for them costs 0.1 us.)
    uint32_t lo = uint32_t(own), hi = uint32_t(own >> 32);
    const bool edges_within = W == 1 || __any((own & ~(uint64_t(1) << lane)) != 0);
    const int here = edges_within ? n - 64 * w : 0;          // rows of this block
#pragma unroll
    for (int k0 = 0; k0 < 32; k0 += 8) {
        if (k0 >= here) break;                               // uniform
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k) {
            const uint32_t row = __builtin_amdgcn_readlane(lo, k);
            lo |= row & uint32_t(__builtin_amdgcn_sbfe(int(lo), k, 1));
        }
    }
#pragma unroll
    for (int k0 = 32; k0 < 64; k0 += 8) {
        if (k0 >= here) break;
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k) {
            const uint32_t row_lo = __builtin_amdgcn_readlane(lo, k), row_hi = __builtin_amdgcn_readlane(hi, k);
            const uint32_t has = uint32_t(__builtin_amdgcn_sbfe(int(hi), k - 32, 1));
            lo |= row_lo & has;
            hi |= row_hi & has;
        }
    }
    own = lo | uint64_t(hi) << 32;
    diagonal[i] = own;
    column[w][i] = own;
    const bool some_more = __any(more);                      // (in all lanes, or lane 0 speaks for itself only)
    if (lane == 0) {
        column[w][kNodes] = 0;
        wave_says[w] = (some_more ? 1 : 0) | (edges_within ? 2 : 0);
    }
    uint64_t *const out = mask + base * words_per_row + w;
    if (i < n) out[int64_t(i) * words_per_row] = own;
    for (int j = lane; j < min(64 * w, n); j += 64) out[int64_t(j) * words_per_row] = 0;          // above the diagonal
    for (int x = W + w; x < words_per_row; x += W)           // words that no node id can reach
        for (int j = lane; j < n; j += 64) mask[(base + j) * words_per_row + x] = 0;
    if (bad && dag_error_flag) *dag_error_flag = 1;
    const int blocks = (n + 63) / 64;
    if (blocks == 1) return;                                 // uniform for the work-group
    __syncthreads();
    int says = 0;
#pragma unroll
    for (int x = 0; x < W; ++x) says |= wave_says[x];
    says = __builtin_amdgcn_readfirstlane(says);
    const bool any_more = says & 1;
    const uint64_t spread = says & 2 ? ~uint64_t(0) : 0;
    int first = 0;
    bool cached = false;
    if (any_more) {                                          // uniform
        first = offset[0];
        const int edges = offset[n] - first;
        cached = edges <= kEdgeCacheInts;
        if (cached)
            for (int e = threadIdx.x; e < edges; e += kNodes) edge_cache[e] = parent_idx[first + e];
        __syncthreads();
    }

    // The blocks below the diagonal, downwards.
    const uint64_t *const mine = column[w];
    for (int c = w + 1; c < blocks; ++c) {
        const int j = 64 * c + lane;
        const uint64_t within = diagonal[j], packed = outer[j];
        uint64_t ext = 0;
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) {
            const int p = int(packed >> (16 * x)) & int(kNone);
            ext |= mine[p != int(kNone) && p >= 64 * w ? p : kNodes];
        }
        if (any_more && j < n) {
            const int e_end = offset[j + 1];
            for (int e = offset[j] + kRegParents; e < e_end; ++e) {
                const int p = cached ? edge_cache[e - first] : parent_idx[e];
                if (p >= 64 * w && p < 64 * c) ext |= mine[p];
            }
        }
        const uint32_t ext_lo = uint32_t(ext), ext_hi = uint32_t(ext >> 32);
        uint32_t row_lo = ext_lo, row_hi = ext_hi;
        const uint64_t from = __ballot(ext != 0) & spread;
        const uint32_t within_lo = uint32_t(within), within_hi = uint32_t(within >> 32);
        // Eight nodes at a time: a layer of a graph is a run of nodes, and with the lanes as constants a node takes five vector
        // instructions and no scalar ones (random graphs, where nearly all have such parents: 2.0 us for 64 nodes one by one).
#pragma unroll
        for (int k0 = 0; k0 < 64; k0 += 8) {
            if (((from >> k0) & 0xff) == 0) continue;        // uniform
#pragma unroll
            for (int k = k0; k < k0 + 8; ++k) {
                const uint32_t has = uint32_t(__builtin_amdgcn_sbfe(int(k < 32 ? within_lo : within_hi), k & 31, 1));
                row_lo |= uint32_t(__builtin_amdgcn_readlane(ext_lo, k)) & has;
                row_hi |= uint32_t(__builtin_amdgcn_readlane(ext_hi, k)) & has;
            }
        }
        const uint64_t row = row_lo | uint64_t(row_hi) << 32;
        column[w][j] = row;
        // the other lanes of the wavefront read it in the next turn: the LDS unit takes its instructions in order
        asm volatile("" ::: "memory");
        if (j < n) out[int64_t(j) * words_per_row] = row;
    }
}

hipError_t launch_build_mask(int32_t batch, int32_t max_nodes, int32_t words_per_row, const int32_t *node_offsets,
                             const int32_t *parent_offsets, const int32_t *parent_idx, uint64_t *mask,
                             int32_t *dag_error_flag, hipStream_t stream) {
    const dim3 grid(batch);
#define GSD_MASK_CASE(WORDS)                                                                                         \
    case WORDS:                                                                                                      \
        hipLaunchKernelGGL(build_mask_kernel<WORDS>, grid, dim3(64 * WORDS), 0, stream, max_nodes, words_per_row, node_offsets,  \
                           parent_offsets, parent_idx, mask, dag_error_flag);                                        \
        break;
    // words computed per row: no node id reaches past word GSD_MAX_NODES_PER_SEQ/64 - 1, wider rows are zero-filled
    static_assert(GSD_MAX_NODES_PER_SEQ == 512, "the cases below cover 512 / 64 = 8 words");
    switch (words_per_row < 8 ? words_per_row : 8) {
        GSD_MASK_CASE(1) GSD_MASK_CASE(2) GSD_MASK_CASE(3) GSD_MASK_CASE(4)
        GSD_MASK_CASE(5) GSD_MASK_CASE(6) GSD_MASK_CASE(7) GSD_MASK_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef GSD_MASK_CASE
    return hipGetLastError();
}

}  // namespace gsd
