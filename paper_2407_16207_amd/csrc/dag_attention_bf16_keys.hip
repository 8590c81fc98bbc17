// bf16 DAG-masked attention for problems with few query rows (paper Sections 4.1 / 5.4), next to the kernel of
// dag_attention_bf16.hip: there the wavefronts of a work-group stand side by side over 128 or 256 rows and walk the keys
// together; here they also stand one behind the other over the keys.
//
// A work-group has RG row groups (head_dim 128: 1 or 2, 64: 1) of 32 rows times four key groups.  A step takes four tiles
// of 32 keys, one per key group: all are copied global -> LDS while the step before is computed, and each wavefront
// computes its 32 rows against its key group's tile with a running maximum of its own (moved only when a row's scores
// exceed it by 2^8).  At the end the four states of a row are merged through LDS.  With fewer rows per work-group there
// are more work-groups, each with fewer steps, and no padding to 128 rows; what a split of the keys over work-groups
// would send through memory and a second launch stays inside the work-group.  (gsd_attn_desc.num_splits still splits on
// top.)
//
// The matrix-core mapping, the swizzles and the copies are those of dag_attention_bf16.hip.  The code is kept small on
// purpose (one rolled loop, a real running maximum instead of the guessed offset and its repair path).
//
// What bounds it: the latency of memory, paid about 1 us at a time, and where the K/V tiles come from (a CU takes in 133 bytes
// per ns from its L2 and all of them together 7 TB/s from the last-level cache).  32 heads of 64 rows over 1088 keys, three splits
// (us inside the kernel): 1.0 until the sequence's offsets are there, 1.3 until all first copies have left, 0.3 until the
// queries have arrived, three steps of 1.0, 0.85 and 0.7 (64 KB each; 1.35 when a step's copies were issued at the start of the step
// before and awaited together), 1.5 to merge and store.  Launch with its merge kernel 14.0 -> 12.3, 24 heads of 64 channels over 5
// ragged sequences of 231 rows 13.9 -> 12.0, 90 rows x 16 heads over 1490 keys 14.1 -> 12.5, a few rows over short contexts 1.1-1.2 times
// as fast.
// Two row groups at head_dim 128 let 64 rows share a tile; at head_dim 64 one row group, of which two work-groups fit a CU (with
// two the best plan over 1000 shapes would be 0.9 % faster).
// Against the better of the other kernel's shapes, before the copies were reordered (merge kernel included, best split count for
// each): 5 ragged sequences of 231 rows, head_dim 64, 15.1 against 17.1 us; 32 heads of 20 rows over 320 keys 9.3-10.0 against 11.6; 192 groups of
// 20 rows, head_dim 64, 10.0 against 13.0; 8 groups of 128 rows over 1056 keys 13.9 against 15.8; behind it from about
// 256 work-groups of 64 rows on (128 groups of 512 rows over 1500 keys 57 against 38).
#include "attention_bf16.h"

namespace gsd {

template <int D, int RG>
struct KeysLds {
    static constexpr int kKeyGroups = 4;
    static constexpr int kRows = RG * 32;
    static constexpr int kTile = 32 * D * 2;                               // bytes of a K or V tile
    static constexpr int kStage = kKeyGroups * 2 * kTile;                  // bytes of a step's tiles
    static constexpr int kOut = kKeyGroups * kRows * D * 4;                // the outputs to be merged take the place of the tiles
    static constexpr int kQ = kOut > 2 * kStage ? kOut : 2 * kStage;       // this step's tiles and the next; then the queries
    static constexpr int kMask = kQ + kRows * D * 2;                       // then the tile's mask words, 16 of 32 bits per node
    static constexpr int kMaskWords = GSD_MAX_NODES_PER_SEQ / 32;
    static constexpr int kTotal = kMask + kRows * kMaskWords * 4;
};

// The LDS is dynamic: from a static size that leaves room for one wave per SIMD the compiler concludes that a wave may have 512
// registers, and then keeps the scores in accumulator registers (32 to 64 moves a step).
template <int D, int RG>
__global__ __launch_bounds__(RG * 256, 2) void dag_attention_bf16_keys_kernel(const AttnParams p) {
    using L = KeysLds<D, RG>;
    constexpr int KG = L::kKeyGroups;
    constexpr int NW = RG * KG;
    constexpr int ROWS = L::kRows;
    constexpr int KS = D / 16;                     // k-steps of S^T = K Q^T
    constexpr int MBD = D / 32;                    // 32-channel blocks of O^T
    constexpr int RB = D * 2;                      // bytes of a K or V row
    constexpr int CHUNKS = D / 8;                  // 16-byte chunks of a row
    constexpr int TB = L::kTile;
    constexpr int STAGE = L::kStage;
    static_assert(D == 128 || RG == 1, "");
    constexpr int RPI = 1024 / RB;                 // rows per wavefront-wide copy
    constexpr int CPW = TB / 1024 / RG;            // copies of K (and of V) per wavefront and step
    constexpr int QPW = ROWS * RB / 1024 / NW;     // copies of the queries per wavefront
    constexpr int MPW = ROWS * L::kMaskWords / 64 / NW;    // and of the mask words, 4 bytes per lane
    static_assert(CPW >= 1 && QPW >= 1 && MPW >= 1, "");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ float m_lds[NW * 32], l_lds[NW * 32];
    auto k_swz = [](int m) __attribute__((always_inline)) -> int { return D == 128 ? (m & 15) : ((m >> 1) & 7); };

    // work-groups of one (sequence, KV head) in consecutive slots of one XCD, see dag_attention_bf16.hip
    const int per_group = p.q_tiles * p.splits;
    const int slot_id = blockIdx.x >> 3;
    const int group_id = (slot_id / per_group) * 8 + (blockIdx.x & 7);
    if (group_id >= p.batch * p.num_kv_heads) return;
    const int within = slot_id % per_group;
    const int qt = within % p.q_tiles, split = within / p.q_tiles;
    const int b = group_id / p.num_kv_heads, kvh = group_id - b * p.num_kv_heads;
    const int32_t node_base = p.node_offsets[b];
    const int32_t n = min(p.node_offsets[b + 1] - node_base, p.max_nodes);
    const int32_t P = p.prefix_lens[b];
    const int64_t kv_elem_off = uniform64(p.kv_offsets[b] * p.kv_ts + int64_t(kvh) * p.kv_hs);
    const int32_t G = p.group;
    const int32_t rows_total = n * G, row0 = qt * ROWS;
    if (row0 >= rows_total) return;                // uniform for the work-group

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = wave % RG, kg = wave / RG;
    const int half = lane >> 5, col = lane & 31;

    const int32_t keys = P + n;
    const int steps_all = (keys + KG * 32 - 1) / (KG * 32);
    const int per_split = (steps_all + p.splits - 1) / p.splits;
    const int s_begin = split * per_split, s_end = min(steps_all, s_begin + per_split);

    // ---- global -> LDS copies: this wavefront's share of its key group's tiles --------------------------------
    const __bf16 *k_seq = p.k + kv_elem_off;
    const __bf16 *v_seq = p.v + kv_elem_off;
    const uint32_t row_stride = uint32_t(p.kv_ts) * 2u;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const uint32_t wave_lds = lds_base + kg * 2 * TB + rg * CPW * 1024;
    const int m0 = rg * CPW * RPI + lane / CHUNKS;             // row position in the tile that copy 0 fills
    const int slot = lane % CHUNKS;
    const uint32_t v_chunk = uint32_t((slot ^ ((CHUNKS / 4) * (m0 & 3))) & (CHUNKS - 1)) * 16u;
    auto copy_k = [&](int s) __attribute__((always_inline)) {
        const int first = (s * KG + kg) * 32;
        const uint32_t to = wave_lds + (s & 1) * STAGE;
#pragma unroll
        for (int j = 0; j < CPW; ++j) {
            const int m = m0 + j * RPI;
            const uint32_t r = uint32_t(min(first + k_lds_row(m), keys - 1));
            dma16_at(k_seq, __umul24(r, row_stride) + uint32_t(slot ^ k_swz(m)) * 16u, to, j * 1024);
        }
    };
    auto copy_v = [&](int s) __attribute__((always_inline)) {
        const int first = (s * KG + kg) * 32;
        const uint32_t to = wave_lds + (s & 1) * STAGE;
#pragma unroll
        for (int j = 0; j < CPW; ++j) {
            const uint32_t r = uint32_t(min(first + m0 + j * RPI, keys - 1));
            dma16_at(v_seq, __umul24(r, row_stride) + v_chunk, to, TB + j * 1024);
        }
    };
    static_assert(RPI % 4 == 0, "v_chunk is the same for all copies of a wavefront");

    // ---- queries and mask words: the same way, ahead of the first V tile ----------------------------------------------
    // Loaded into registers they would be awaited by the compiler, which does not count the copies and would wait for all of
    // them.  Queries lie like K rows, chunk x of row r in slot x ^ k_swz(r); of the mask the words of the tile's nodes.
    const int32_t first_node = row0 / G, last_node = min(row0 + ROWS - 1, rows_total - 1) / G;
    if (s_begin < s_end) {
        copy_k(s_begin);                           // first: the addresses of the others take a while
#pragma unroll
        for (int j = 0; j < QPW; ++j) {
            const int m = (wave * QPW + j) * RPI + lane / CHUNKS;
            const int32_t r = min(row0 + m, rows_total - 1), node = r / G;
            dma16_from(p.q + (int64_t(node_base) + node) * p.q_ts + int64_t(kvh * G + r - node * G) * p.q_hs + (slot ^ k_swz(m)) * 8,
                       lds_base + L::kQ + (wave * QPW + j) * 1024);
        }
#pragma unroll
        for (int j = 0; j < MPW; ++j) {
            const int x = (wave * MPW + j) * 64 + lane;
            const int32_t node = min(first_node + x / L::kMaskWords, last_node);
            const int word = min(x % L::kMaskWords, 2 * p.words_per_row - 1);
            dma4_from(reinterpret_cast<const uint32_t *>(p.mask + (int64_t(node_base) + node) * p.words_per_row) + word,
                      lds_base + L::kMask + (wave * MPW + j) * 256);
        }
        copy_v(s_begin);
        if (RG == 1 && s_begin + 1 < s_end) copy_k(s_begin + 1);
    }
    const int32_t my_row = min(row0 + rg * 32 + col, rows_total - 1);
    const uint32_t *my_mask = reinterpret_cast<const uint32_t *>(lds + L::kMask) + (my_row / G - first_node) * L::kMaskWords;

    floatx16 acc[MBD];
#pragma unroll
    for (int x = 0; x < MBD; ++x)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[x][j] = 0.f;
    float m = kMInit, l = 0.f;                     // running maximum (log2 domain) and this half's share of the sum
    const float c = p.scale_log2e;

    // ---- LDS read addresses, see dag_attention_bf16.hip ---------------------------------------------------------
    uint32_t k_off[KS], v_off[MBD];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        k_off[ks] = (uint32_t(col * RB + ((half ^ k_swz(col)) * 16)) ^ uint32_t(ks * 32)) + uint32_t(kg * 2 * TB);
    {
        const int sl = lane & 15, grp = lane >> 4;
        const int y = (grp & 1) * 2 + (sl & 3) / 2;
        const uint32_t v0 = uint32_t((8 * (grp >> 1) + sl / 4) * RB + (((y ^ ((CHUNKS / 4) * (sl / 4))) & (CHUNKS - 1)) * 16) +
                                     (sl & 1) * 8);
#pragma unroll
        for (int x = 0; x < MBD; ++x) v_off[x] = (v0 ^ uint32_t(x * 64)) + uint32_t(kg * 2 * TB + TB);
    }
    bf16x8 qf[KS];
    if (s_begin < s_end) {
        // the queries, the mask words and the first K tile are older than the copies that may stay in flight
        if (RG == 1 && s_begin + 1 < s_end) dma_wait<2 * CPW>();
        else dma_wait<CPW>();
        wg_barrier();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(lds + L::kQ + rg * 32 * RB + (k_off[ks] - kg * 2 * TB));
    }

    // Step s: scores from K(s), then P.V from V(s).
    // With one row group a tile belongs to one wavefront, which has nobody to meet: V(s+1) is fetched from the top of the step
    // on, K(s+2) from where K(s) has been read, so that one and a half to two steps' tiles are on their way at any time.
    // With two, two wavefronts copy a half of a tile each and read both, and share a SIMD with two others: one barrier a step, at
    // which the whole next step is fetched (the finer order above with its two barriers took 7 % longer).
    for (int s = s_begin; s < s_end; ++s) {
        const bool more = s + 1 < s_end;
        if (RG > 1) dma_wait<0>();                               // K(s) and V(s) have landed
        else if (more) dma_wait<2 * CPW>();                      // K(s) has; behind it V(s) and K(s+1) may be on their way
        else dma_wait<CPW>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the tiles of step s-1 have been read
        if (RG > 1) wg_barrier();
        if (RG > 1 && more) copy_k(s + 1);
        if (more) copy_v(s + 1);
        const int first = (s * KG + kg) * 32;
        uint32_t bits = ~0u;
        if (first + 32 > P) {                      // uniform: the tile reaches into the draft nodes
            const int32_t pos = first - P;         // its first key's draft node; below 0: prefix, 32 visible keys
            const int32_t w = min((pos + 32) >> 5, L::kMaskWords), left = n - pos;
            const uint32_t lo = w == 0 ? ~0u : my_mask[w - 1], hi = my_mask[min(w, L::kMaskWords - 1)];
            bits = uint32_t(((uint64_t(hi) << 32) | lo) >> (pos & 31));
            if (left < 32) bits &= left > 0 ? (1u << left) - 1 : 0u;
        }
        const bool seen = __any(bits != 0);        // uniform; else no row of the wavefront sees a key of the tile
        const char *tile = lds + (s & 1) * STAGE;
        floatx16 sc;
        if (seen) {
            bf16x8 kf[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8 *>(tile + k_off[ks]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 16; ++j) sc[j] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sc, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (RG == 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // K(s) has been read
            if (s + 2 < s_end) {
                copy_k(s + 2);
                dma_wait<3 * CPW>();               // V(s) has landed; behind it K(s+1), V(s+1), K(s+2)
            } else if (more) {
                dma_wait<2 * CPW>();
            } else {
                dma_wait<0>();
            }
        }
        if (seen) {
            bf16x8 vf[2][MBD];
            auto read_v = [&](int ks2) __attribute__((always_inline)) {
#pragma unroll
                for (int x = 0; x < MBD; ++x) {
                    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
                    const char *at = tile + ks2 * 16 * RB + v_off[x];
                    const uint32_t at_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)at;
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(uintptr_t)at_lds);
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(uintptr_t)(at_lds + 4 * RB));
                    vf[ks2][x] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            };
            read_v(0);
            read_v(1);
            __builtin_amdgcn_sched_barrier(0);
            if (first + 32 > P) {                  // register i is key 16*(i/8) + 8*half + i%8
                const uint32_t mine = bits >> (8 * half);
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (!((mine >> (16 * (i / 8) + i % 8)) & 1)) sc[i] = -__builtin_inff();
            }
            float mx = fmaxf(sc[0], sc[1]);
#pragma unroll
            for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(sc[i], sc[i + 1]));
            // the maximum only has to be near: rows are moved to a new one when some row's scores exceed the old by 2^8
            const float m_new = fmaxf(m, max_across_halves(mx) * c);
            if (__any(m_new > m + 8.f)) {
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                l *= alpha;
#pragma unroll
                for (int x = 0; x < MBD; ++x)
#pragma unroll
                    for (int j = 0; j < 16; ++j) acc[x][j] *= alpha;
                m = m_new;
            }
            u32x4 pf[2];
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                floatx2 x;
                x[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i], c, -m));
                x[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i + 1], c, -m));
                l += x[0] + x[1];
                pf[i / 8][(i / 2) % 4] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
            }
#pragma unroll
            for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
                for (int x = 0; x < MBD; ++x)
                    acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks2][x], __builtin_bit_cast(bf16x8, pf[ks2]), acc[x], 0, 0, 0);
        }
    }

    // ---- merge of the KG states of every row ------------------------------------------------------------------
    // accumulator register i of channel block x is channel x*32 + 8*(i/4) + 4*half + i%4; 16-byte chunks of the fp32
    // rows are XOR-swizzled by the row
    {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        if (half == 0) {
            m_lds[kg * ROWS + rg * 32 + col] = m;
            l_lds[kg * ROWS + rg * 32 + col] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
    }
    __syncthreads();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    {
        float top = m_lds[rg * 32 + col];
#pragma unroll
        for (int g = 1; g < KG; ++g) top = fmaxf(top, m_lds[g * ROWS + rg * 32 + col]);
        const float f = __builtin_amdgcn_exp2f(m - top);
        floatx4 *out = reinterpret_cast<floatx4 *>(lds) + (kg * ROWS + rg * 32 + col) * (D / 4);
#pragma unroll
        for (int x = 0; x < MBD; ++x)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                floatx4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = acc[x][4 * i4 + e] * f;
                out[(x * 8 + 2 * i4 + half) ^ (col & (D / 4 - 1))] = y;
            }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < ROWS * (D / 8); idx += NW * 64) {
        const int row = idx / (D / 8), chunk = idx - row * (D / 8);          // 8 channels
        if (row0 + row >= rows_total) break;                                   // rows ascend with idx
        float top = m_lds[row], sum = 0.f;
#pragma unroll
        for (int g = 1; g < KG; ++g) top = fmaxf(top, m_lds[g * ROWS + row]);
        floatx4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            sum += l_lds[g * ROWS + row] * __builtin_amdgcn_exp2f(m_lds[g * ROWS + row] - top);
            const floatx4 *from = reinterpret_cast<const floatx4 *>(lds) + (g * ROWS + row) * (D / 4);
            y0 += from[(2 * chunk) ^ (row & 31 & (D / 4 - 1))];
            y1 += from[(2 * chunk + 1) ^ (row & 31 & (D / 4 - 1))];
        }
        const int32_t node = (row0 + row) / G, head = kvh * G + (row0 + row - node * G);
        const int64_t t = int64_t(node_base) + node;
        if (p.splits == 1) {
            const float inv = sum > 0.f ? 1.f / sum : 0.f;
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] = (__bf16)(y0[e] * inv);
                o[4 + e] = (__bf16)(y1[e] * inv);
            }
            *reinterpret_cast<bf16x8 *>(p.o + t * p.o_ts + int64_t(head) * p.o_hs + 8 * chunk) = o;
            if (p.lse && chunk == 0)
                p.lse[t * p.num_q_heads + head] = sum > 0.f ? (top + __log2f(sum)) * 0.6931471805599453f : -__builtin_inff();
        } else {
            const int64_t prow = (int64_t(split) * p.total_nodes + t) * p.num_q_heads + head;
            floatx4 *part = reinterpret_cast<floatx4 *>(p.part_o + prow * D + 8 * chunk);
            part[0] = y0;
            part[1] = y1;
            if (chunk == 0) {
                floatx2 ml;
                ml[0] = top;
                ml[1] = sum;
                *reinterpret_cast<floatx2 *>(p.part_ml + prow * 2) = ml;
            }
        }
    }
}

hipError_t launch_attention_bf16_keys(const AttnParams &p, int head_dim, int row_groups, hipStream_t stream) {
    const dim3 grid((unsigned)(p.wg_per_xcd * 8)), block(row_groups * 256);
    if (head_dim == 128) {
        if (row_groups == 1)
            hipLaunchKernelGGL((dag_attention_bf16_keys_kernel<128, 1>), grid, block, (KeysLds<128, 1>::kTotal), stream, p);
        else
            hipLaunchKernelGGL((dag_attention_bf16_keys_kernel<128, 2>), grid, block, (KeysLds<128, 2>::kTotal), stream, p);
    } else {
        hipLaunchKernelGGL((dag_attention_bf16_keys_kernel<64, 1>), grid, block, (KeysLds<64, 1>::kTotal), stream, p);
    }
    return hipGetLastError();
}

}  // namespace gsd
