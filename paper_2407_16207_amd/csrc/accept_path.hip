// Longest accepted root path per sequence (deterministic verification, paper Sections 3 and 4.1).
//
// An edge p -> i is accepted iff tokens[i] equals the LLM's choice after p (pred[p], or root_pred for the
// root); the first mismatch on a hypothesis discards everything after it, and the longest accepted path from
// the root is taken.  One work-group per sequence: L[i] (nodes on the longest accepted root path ending at i,
// -1 if none) is relaxed over all nodes in parallel until it stops changing (hard bound = node count), then the best end
// node is reduced and one thread walks the back-pointers.  Ties: smallest end node id, then the smallest-id qualifying parent.
#include "gsd_internal.h"

namespace gsd {

constexpr int kAcceptEdgeCache = 6144;         // parent entries of a sequence that LDS has room for

template <int THREADS>
__global__ __launch_bounds__(THREADS) void accept_kernel(
    int32_t max_nodes, const int32_t *__restrict__ node_offsets, const int32_t *__restrict__ parent_offsets,
    const int32_t *__restrict__ parent_idx, const int32_t *__restrict__ tokens, const int32_t *__restrict__ pred,
    const int32_t *__restrict__ root_pred, int32_t *__restrict__ accept_len, int32_t *__restrict__ accept_path,
    int32_t *__restrict__ bonus_token) {
    __shared__ int32_t L[THREADS];
    __shared__ int32_t pred_s[THREADS];
    __shared__ int32_t path_s[THREADS];
    __shared__ int32_t back_s[THREADS];
    __shared__ int32_t edge_s[kAcceptEdgeCache];
    __shared__ uint32_t wave_best[THREADS / 64];
    __shared__ int32_t grew_s[3];                  // of a round of the relaxation: some L has grown
    __shared__ int32_t len_s;

    const int b = blockIdx.x;
    const int64_t base = node_offsets[b];
    int n = node_offsets[b + 1] - node_offsets[b];
    if (n > max_nodes) n = max_nodes;
    if (n < 0) n = 0;
    const int32_t rp = root_pred[b];
    const int32_t e_first = parent_offsets[base];

    // One thread per node (the launcher: THREADS >= max_nodes).  Whether an edge is accepted never changes, so it is decided
    // once; the first four parents of a node, fetched together with clamped indices instead of branches, stay in registers,
    // which leaves a sweep with four independent LDS reads and no branch per parent (branches serialise the round trips).
    constexpr int kRegParents = 4;
    const int i = threadIdx.x;
    const bool active = i < n;
    int par[kRegParents];          // parent id; -1 = root; -2 = no such edge, or not accepted
    int e_lo = 0, e_hi = 0;
    int32_t my_tok = 0;
#pragma unroll
    for (int x = 0; x < kRegParents; ++x) par[x] = -2;
    // is edge p -> i accepted (p is a well-formed parent of i)?
    auto accepted = [&](int p) -> bool { return my_tok == (p == -1 ? rp : pred_s[p]); };
    if (active) {
        e_lo = parent_offsets[base + i];
        e_hi = parent_offsets[base + i + 1];
        my_tok = tokens[base + i];
        pred_s[i] = pred[base + i];
        L[i] = -1;
        if (e_hi > e_lo) {
#pragma unroll
            for (int x = 0; x < kRegParents; ++x) par[x] = parent_idx[min(e_lo + x, e_hi - 1)];
        }
    }
    if (i < 3) grew_s[i] = 0;
    __syncthreads();
    if (active) {
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) {
            const int p = par[x];
            const bool edge = e_lo + x < e_hi && p >= -1 && p < i;
            const int32_t llm = pred_s[edge && p >= 0 ? p : i];
            par[x] = edge && my_tok == (p == -1 ? rp : llm) ? p : -2;
        }
    }
    // Rare: a node with more than four parents.  Those of the others that are accepted go to its place in LDS, once, and the
    // sweeps look at nothing else.  8 sequences of 512 nodes with up to 20 parents: 91 us, 170 with every entry read from memory
    // and decided again in every sweep (as lists beyond the LDS room still are: up to 40 parents, 594 us), 167 with a copy
    // of all lists in LDS, decided in every sweep.  4 parents at most: nothing (6.2 us either way).
    const bool more = active && e_hi - e_lo > kRegParents;
    const bool in_lds = more && e_lo >= e_first && e_hi - e_first <= kAcceptEdgeCache;
    int32_t *const kept = edge_s + (in_lds ? e_lo - e_first : 0);
    int kept_count = 0;
    // every further parent of this node whose edge is accepted, handed to f in the order of the list
    auto each_further = [&](auto &&f) {
        constexpr int kBatch = 8;
        for (int e0 = e_lo + kRegParents; e0 < e_hi; e0 += kBatch) {
            int p[kBatch];
#pragma unroll
            for (int x = 0; x < kBatch; ++x) p[x] = parent_idx[min(e0 + x, e_hi - 1)];
#pragma unroll
            for (int x = 0; x < kBatch; ++x)
                if (e0 + x < e_hi && p[x] >= -1 && p[x] < i && accepted(p[x])) f(p[x]);
        }
    };
    if (in_lds) each_further([&](int p) { kept[kept_count++] = p; });
    auto each_accepted = [&](auto &&f) {
        if (in_lds)
            for (int x = 0; x < kept_count; ++x) f(kept[x]);
        else
            each_further(f);
    };

    // L only grows and whatever is read is the length of a path that exists, so a wavefront follows its own nodes until
    // they rest or for a few steps, and the wavefronts then meet to find out whether all rest (one alone does not have to meet).
    // A wavefront that has to look at further parents takes one step at a time.  Launches in a replayed graph, against a sweep
    // with a barrier and a reduction for every step (us): 64 nodes 3.2-5.3 -> 3.1-4.65, 8 x 256 of <= 3 parents 5.2-8.7 -> 4.7-6.6,
    // 32 x 512 6.7-10.8 -> 5.8-9.2 (the longer times: paths of more than a dozen nodes are accepted).
    constexpr bool kAlone = THREADS == 64;
    const int steps = kAlone ? n + 1 : __any(more) ? 1 : 4;
    int32_t mine = -1;             // L[i]
    for (int round = 0; round <= n; ++round) {
        bool grew = false;
        for (int step = 0; step < steps; ++step) {
            bool up = false;
            if (active) {
                int32_t best = mine;
#pragma unroll
                for (int x = 0; x < kRegParents; ++x) {
                    const int32_t l = __hip_atomic_load(&L[par[x] >= 0 ? par[x] : i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const int32_t lp = par[x] >= 0 ? l : (par[x] == -1 ? 0 : -1);
                    if (lp >= 0 && lp + 1 > best) best = lp + 1;
                }
                if (more) {
                    each_accepted([&](int p) {
                        const int32_t lp = p == -1 ? 0 : __hip_atomic_load(&L[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (lp >= 0 && lp + 1 > best) best = lp + 1;
                    });
                }
                up = best != mine;
                if (up) {
                    mine = best;
                    __hip_atomic_store(&L[i], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            if (!__any(up)) break;
            grew = true;
        }
        if (kAlone) break;
        // three flags in turn: one is written, one read, and the one that everybody has read is cleared
        const int at = round % 3;
        if (grew) grew_s[at] = 1;
        __syncthreads();
        if (i == 0) grew_s[(round + 2) % 3] = 0;
        if (grew_s[at] == 0) break;
    }

    // back pointer of every accepted node: the smallest-id accepted parent that ends a path one node shorter
    // (the root, id -1, is the smallest)
    if (active && mine > 0) {
        int32_t chosen = 0x7fffffff;
#pragma unroll
        for (int x = 0; x < kRegParents; ++x) {
            const int32_t l = L[par[x] >= 0 ? par[x] : i];
            const int32_t lp = par[x] >= 0 ? l : (par[x] == -1 ? 0 : -1);
            if (lp == mine - 1 && par[x] < chosen) chosen = par[x];
        }
        if (more) {
            each_accepted([&](int p) {
                const int32_t lp = (p == -1) ? 0 : L[p];
                if (lp == mine - 1 && p < chosen) chosen = p;
            });
        }
        back_s[i] = chosen;
    }

    // best end node: largest L, then smallest id.  key = L * 1024 + (1023 - i), 0 = nothing accepted.
    uint32_t key = 0;
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
        len_s = len;
        accept_len[b] = len;
        bonus_token[b] = (len > 0) ? pred_s[v] : rp;
        for (int pos = len - 1; pos >= 0 && v >= 0 && v < n; --pos) {   // L drops by one per step: the root's child sits at pos 0
            path_s[pos] = v;
            v = back_s[v];
        }
    }
    __syncthreads();
    const int32_t len = len_s;
    int32_t *out = accept_path + int64_t(b) * max_nodes;
    for (int x = threadIdx.x; x < max_nodes; x += THREADS) out[x] = (x < len) ? path_s[x] : -1;
}

hipError_t launch_accept(int32_t batch, int32_t max_nodes, const int32_t *node_offsets,
                         const int32_t *parent_offsets, const int32_t *parent_idx, const int32_t *tokens,
                         const int32_t *pred, const int32_t *root_pred, int32_t *accept_len, int32_t *accept_path,
                         int32_t *bonus_token, hipStream_t stream) {
    // The fewest wavefronts that hold a node per lane: each more costs the launch and every barrier of the sweeps.
    // 64 nodes: 3.4 us with one, 4.5 with eight and the parents
    // passed through LDS first; 8 sequences of 256: 6.1 against 6.8 us; 32 of 512: 9.7 against 10.8.
#define GSD_ACCEPT(THREADS)                                                                                          \
    hipLaunchKernelGGL(accept_kernel<THREADS>, dim3(batch), dim3(THREADS), 0, stream, max_nodes, node_offsets,       \
                       parent_offsets, parent_idx, tokens, pred, root_pred, accept_len, accept_path, bonus_token)
    static_assert(GSD_MAX_NODES_PER_SEQ == 512, "the cases below cover 512 nodes");
    if (max_nodes <= 64) GSD_ACCEPT(64);
    else if (max_nodes <= 128) GSD_ACCEPT(128);
    else if (max_nodes <= 256) GSD_ACCEPT(256);
    else GSD_ACCEPT(512);
#undef GSD_ACCEPT
    return hipGetLastError();
}

}  // namespace gsd
