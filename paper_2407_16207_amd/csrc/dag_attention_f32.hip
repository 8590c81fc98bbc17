// fp32 DAG-masked attention (paper Sections 4.1 / 5.4): the full-precision variant, on the fp32 matrix instructions.
//
// The G query heads of a KV head share K/V, so the (node, head) pairs of one (sequence, KV head) are packed into one
// row space r = node*G + g and cut into tiles of 16 rows.  A work-group of 4 wavefronts owns one tile; the keys
// [prefix ; draft nodes] are dealt to the wavefronts in runs of 16 (wavefront w takes runs w, w+4, ...), each keeps its
// own running (max, sum, output) and the four states are merged through LDS at the end.
//
// v_mfma_f32_16x16x4_f32 (fp32 products, fp32 accumulation).  Scores are computed transposed, S^T = K Q^T: a lane owns
// one query row (column l%16) and the four keys 4*(l/16)+r, and exactly these four registers are the B operands of the
// second contraction O^T += V^T P^T when its step r is fed with the V rows 4*(l/16)+r: nothing is exchanged between
// lanes.  Loads follow memory, not operands: neighbouring lanes fetch neighbouring 16-byte chunks of a row.  For V that
// is an operand layout (the order of the output channels is free); K goes through a part of LDS that is the
// wavefront's own (loaded in operand layout, a line per lane: 32.6 us instead of 30.0 on the case below).  The next V
// and K runs are in flight while the matrix instructions of a run execute.
//
// What bounds it: a SIMD's matrix and vector instructions one after the other (a second wavefront per SIMD hides
// nothing: 8 wavefronts over the same tiles take the same time), 64 matrix instructions of 14 ns per run at head_dim
// 128 and a third of that again for softmax and addresses; with fewer tiles than CUs, the idle CUs.
// 32 heads of 64 rows over 1088 keys, head_dim 128 (128 tiles, half the chip): 31.4 us = 36 TFLOP/s; 8 groups of 960
// rows over 1120 keys: 53 us = 78 TFLOP/s of the 154 that a large fp32 matrix product reaches.  The plain-FMA kernel
// before this one (a lane per key, every lane reading a K and a V row of its own) took 313 and 1147 us, and 24.8 us
// where this one takes 7.1 (4 heads, 16 nodes, 144 keys, head_dim 64).
// Summed in one level the outputs were further from 64-bit sums than that kernel's (relative 4.5e-7 against 4.1e-7 on the
// first case, 5.1e-7 against 3.6e-7 at head_dim 64); in two levels, with two chains per score, they are nearer (3.2e-7 and
// 3.0e-7), for about 1 us.
// 32-row tiles (every K/V operand used twice) need 232 registers and lose more to the coarser split: 51 and 54 us.
// With a workspace the keys are also split over work-groups where the tiles leave CUs idle (attention_f32_splits), merged
// by the kernel that merges the bf16 splits: the 128 tiles above then take 23.5 us, merge included.
// Since then a turn of the four wavefronts (16 keys each) takes 1.47 us instead of 1.73, 0.9 of them its matrix instructions: K operands
// read from LDS a pair ahead, 32-bit offsets to scalar bases, rows moved to a new maximum only where it exceeds the old by
// 2^3, first tiles fetched ahead of the mask words.  The same case 24.6 -> 23.1 us (replayed), 64 heads of 16 nodes over 1852 keys, 3
// sequences, 31.7 -> 27.5, 8 of 319 rows over 1238 keys 33.2 -> 30.3; 50 random shapes 0.995-1.155 times as fast; the relative
// error against 64 bits is what it was (2.0-3.4e-7 over 14 shapes, each within 0.5 % of before).
#include "attention_bf16.h"

namespace gsd {

namespace {

constexpr int kF32Waves = 4;
constexpr float kF32Log2e = 1.4426950408889634f;
constexpr float kF32Empty = -1e30f;      // running max before any visible key; finite, so that differences stay numbers

struct F32Params {
    const float *q;
    float *o;
    float *lse;
    const float *k;
    const float *v;
    const int64_t *kv_offsets;
    const int32_t *prefix_lens;
    const int32_t *node_offsets;
    const uint64_t *mask;
    int64_t q_ts, q_hs, o_ts, o_hs, kv_ts, kv_hs;
    float *part_o, *part_ml;             // as in AttnParams; used if splits > 1
    int64_t part_rows;                   // total_nodes * num_q_heads
    int32_t groups, max_nodes, num_q_heads, num_kv_heads, group, words_per_row, row_tiles, splits;
    float scale_log2e;
};

// max over the four 16-lane groups of a wavefront (lanes l, l^16, l^32, l^48), in every lane
__device__ __forceinline__ float max_across_groups(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_across_groups(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Offset: type of the byte offsets within a run of 16 K/V rows.  32 bits let the loads take their base from scalar registers (64-bit
// offsets cost two registers and an addition per load); row strides that do not fit get 64.  (Rows 128 MiB apart: at head_dim 128
// that spills four registers, 4 heads of 16 nodes over 256 keys 11.5 us where the kernel without K operands ahead took 11.2.)
template <int D, typename Offset>
__global__ __launch_bounds__(kF32Waves * 64, 2) void dag_attention_f32_kernel(const F32Params p) {
    constexpr int NW = kF32Waves;
    constexpr int KV4 = D / 16;           // float4 loads of a K row fragment (4 channels per lane and load)
    constexpr int CB = D / 16;            // 16-channel blocks of the output
    constexpr int VV4 = CB / 4;           // float4 loads per V row and lane
    constexpr int ROWS = 16;
    constexpr int CHUNKS = D / 4;         // 16-byte chunks of an output row
    __shared__ __attribute__((aligned(16))) float o_lds[NW * ROWS * D];
    constexpr int kMaskWords = GSD_MAX_NODES_PER_SEQ / 64;
    __shared__ uint64_t mask_lds[ROWS][kMaskWords + 1];
    __shared__ float m_lds[NW * ROWS], l_lds[NW * ROWS];

    // the row tiles of one (sequence, KV head) share K/V: they take consecutive slots of one XCD (ids are dealt
    // round-robin to the 8 XCDs), the (sequence, KV head) groups go round the XCDs
    const int slot = blockIdx.x >> 3, per_group = p.row_tiles * p.splits;
    const int group_id = (slot / per_group) * 8 + (blockIdx.x & 7);
    const int split = slot % per_group / p.row_tiles;    // the row tiles of a split are neighbours
    if (group_id >= p.groups) return;
    const int b = group_id / p.num_kv_heads, kvh = group_id - b * p.num_kv_heads;
    const int32_t node_base = p.node_offsets[b];
    const int32_t n = min(p.node_offsets[b + 1] - node_base, p.max_nodes);
    const int32_t P = p.prefix_lens[b];
    const int64_t kv_row0 = p.kv_offsets[b];
    const int32_t G = p.group;
    const int32_t rows_total = n * G, row0 = (slot % p.row_tiles) * ROWS;
    if (row0 >= rows_total) return;                      // uniform for the work-group

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, kg = lane >> 4;
    const int32_t keys = P + n, all_tiles = (keys + 15) / 16, per_split = (all_tiles + p.splits - 1) / p.splits;
    const int32_t first = split * per_split, tiles = min(all_tiles, first + per_split);     // this split's; may be none
    // K rows come whole (neighbouring lanes, neighbouring 16-byte chunks) into registers, go from there to a part of LDS
    // that is this wavefront's own and are read back as operands: lane l holds row l%16, and loads that follow the
    // operand layout touch a line per lane.  Chunk x of row r sits in slot x ^ r: the 16 rows meet in no bank.
    // V operands are D/16 channels of a row per lane, neighbouring lanes side by side: loaded as they are.
    constexpr int KROWS = 64 / CHUNKS;                   // K rows per load
    const float *kv_base_k = p.k + kv_row0 * p.kv_ts + kvh * p.kv_hs, *kv_base_v = p.v + kv_row0 * p.kv_ts + kvh * p.kv_hs;
    const int k_row = lane / CHUNKS, k_chunk = lane % CHUNKS;
    floatx4 ks[KV4], vf[4][VV4];
    Offset k_off[KV4], v_off[4];                         // bytes from the tile's first row
    const Offset row_bytes = Offset(p.kv_ts * 4);
    auto set_offsets = [&](int last) __attribute__((always_inline)) {     // rows past `last` repeat it
#pragma unroll
        for (int j = 0; j < KV4; ++j) k_off[j] = Offset(min(j * KROWS + k_row, last)) * row_bytes + 16 * k_chunk;
#pragma unroll
        for (int r = 0; r < 4; ++r) v_off[r] = Offset(min(4 * kg + r, last)) * row_bytes + 16 * col;
    };
    set_offsets(15);
    auto load_k = [&](int tile) __attribute__((always_inline)) {          // past the last tile: loads that nothing waits for
        const int t = min(tile, tiles - 1);
        if (t * 16 + 16 > keys) set_offsets(keys - 1 - t * 16);           // uniform; no full tile comes after it
        const char *base = reinterpret_cast<const char *>(kv_base_k + int64_t(t) * 16 * p.kv_ts);
#pragma unroll
        for (int j = 0; j < KV4; ++j) ks[j] = *reinterpret_cast<const floatx4 *>(base + k_off[j]);
    };
    auto load_v = [&](int tile) __attribute__((always_inline)) {          // after load_k of the same tile
        const char *base = reinterpret_cast<const char *>(kv_base_v + int64_t(min(tile, tiles - 1)) * 16 * p.kv_ts);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < VV4; ++t) vf[r][t] = *reinterpret_cast<const floatx4 *>(base + v_off[r] + 256 * t);
    };
    floatx4 *my_k = reinterpret_cast<floatx4 *>(o_lds) + wave * 16 * CHUNKS;
    auto store_k = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < KV4; ++j) {
            const int r = j * KROWS + k_row;
            my_k[r * CHUNKS + (k_chunk ^ r)] = ks[j];
        }
    };

    load_k(first + wave);                                // ahead of the mask words, which are waited for on their way into LDS
    load_v(first + wave);

    // Sums in two levels, or their rounding errors would grow with the length of the context: the running ones take
    // kFold tiles and are then added to the totals.
    constexpr int kFold = 8;
    floatx4 qf[KV4], acc[CB], total[CB];
    float m = kF32Empty, l = 0.f, l_total = 0.f;
    const int32_t q_row = min(row0 + col, rows_total - 1), q_node = q_row / G;
    const float *qp = p.q + (int64_t(node_base) + q_node) * p.q_ts + (kvh * G + (q_row - q_node * G)) * p.q_hs + 4 * kg;
#pragma unroll
    for (int t = 0; t < KV4; ++t) qf[t] = *reinterpret_cast<const floatx4 *>(qp + 16 * t);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = total[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            total[cb] += acc[cb];
            acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        l_total += l;
        l = 0.f;
    };
    // the words of the tile's mask rows in LDS: fetched inside the loop they would queue behind the K/V loads in flight
    for (int x = threadIdx.x; x < ROWS * kMaskWords; x += NW * 64) {
        const int row = x / kMaskWords, w = x - row * kMaskWords;
        const int32_t node = min(row0 + row, rows_total - 1) / G;
        mask_lds[row][w + 1] = w < p.words_per_row ? p.mask[(int64_t(node_base) + node) * p.words_per_row + w] : 0;
        if (w == 0) mask_lds[row][0] = ~uint64_t(0);     // the keys before draft node 0: the end of the prefix
    }
    const float c = p.scale_log2e;
    store_k();
    __syncthreads();

    // K operands are read from LDS one pair of 16-channel groups ahead of the matrix instructions that take them, the first pair of a
    // run behind the stores of the run before.
    floatx4 kf[2][2];
    auto read_k = [&](int pair) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2; ++x) kf[pair & 1][x] = my_k[col * CHUNKS + ((4 * (2 * pair + x) + kg) ^ col)];
    };
    read_k(0);

    int left = kFold;                                    // tiles until the next fold
    bool spoiled = false;                                // uniform: a V element that is no finite number was left out
    for (int tile = first + wave; tile < tiles; tile += NW) {
        load_k(tile + NW);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 s = {0.f, 0.f, 0.f, 0.f}, s_odd = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int pair = 0; pair < KV4 / 2; ++pair) {
            if (pair + 1 < KV4 / 2) read_k(pair + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[pair & 1][0][e], qf[2 * pair][e], s, 0, 0, 0);
                s_odd = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[pair & 1][1][e], qf[2 * pair + 1][e], s_odd, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        s += s_odd;
        if (tile * 16 + 16 > P) {                        // uniform: the tile reaches into the draft nodes
            const int32_t pos = tile * 16 + 4 * kg - P;  // draft node of this lane's first key; below 0: prefix
            constexpr int32_t kLastWord = 2 * kMaskWords + 1;     // beyond it: keys past the end, dropped by pos + r >= n
            const int32_t w = min((pos + 64) >> 5, kLastWord);    // its 32-bit word of the row in LDS, >= 1
            const uint32_t *words = reinterpret_cast<const uint32_t *>(mask_lds[col]);
            const uint32_t lo = words[w], hi = words[min(w + 1, kLastWord)];
            const uint32_t bits = uint32_t(((uint64_t(hi) << 32) | lo) >> (pos & 31));
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (!((bits >> r) & 1) || pos + r >= n) s[r] = -__builtin_inff();
        }
        const float mx = max_across_groups(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
        const float m_new = fmaxf(m, mx * c);
        // Rows are moved to a new maximum when some row's scores exceed the old by 2^3: probabilities up to 8 lose nothing, and
        // with 16 rows there is a new maximum in most tiles, 66 multiplications each.
        if (__any(m_new > m + 3.f)) {            // uniform
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);
            l *= alpha;
            l_total *= alpha;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                acc[cb] *= alpha;
                total[cb] *= alpha;
            }
            m = m_new;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -m));
            l += s[r];
        }
        if (tile * 16 + 16 > P) {                        // uniform, as above: a key may be hidden from some rows of the tile
            float top[2] = {0.f, 0.f};                   // largest magnitude, NaN if there is one: two values per instruction
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < VV4; ++t)
#pragma unroll
                    for (int e = 0; e < 4; e += 2)
                        top[e / 2] = __builtin_elementwise_maximum(
                            __builtin_elementwise_maximum(top[e / 2], fabsf(vf[r][t][e])), fabsf(vf[r][t][e + 1]));
            if (__any(!(__builtin_elementwise_maximum(top[0], top[1]) < __builtin_inff()))) {
                // times a hidden key's 0 such an element would be a NaN for rows that must not see it; what those who see
                // it get of it is added after the loop (the search costs nothing on the first case above, 2 % without prefix)
                spoiled = true;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int t = 0; t < VV4; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (!(fabsf(vf[r][t][e]) < __builtin_inff())) vf[r][t][e] = 0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][cb / 4][cb % 4], s[r], acc[cb], 0, 0, 0);
        store_k();
        read_k(0);
        load_v(tile + NW);
        if (--left == 0) {                               // uniform
            fold();
            left = kFold;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    fold();
    // V elements that are no finite numbers, left out above in the tiles that reach into the draft nodes: a row that sees
    // the key ends up with them whatever else it sums.  Register i of channel block 4*x + e is channel 64*x + 16*kg + 4*i + e.
    if (spoiled) {
        for (int tile = first + wave; tile < tiles; tile += NW) {
            if (tile * 16 + 16 <= P) continue;
            for (int key = tile * 16; key < min(tile * 16 + 16, keys); ++key) {
                const int32_t pos = key - P;
                const bool seen = pos < 0 || ((mask_lds[col][1 + (pos >> 6)] >> (pos & 63)) & 1);
                const float *at = kv_base_v + key * p.kv_ts + 16 * kg;
#pragma unroll
                for (int x = 0; x < VV4; ++x)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const floatx4 v = *reinterpret_cast<const floatx4 *>(at + 64 * x + 4 * i);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (seen && !(fabsf(v[e]) < __builtin_inff())) total[4 * x + e][i] += v[e];
                    }
            }
        }
    }

    __syncthreads();                                     // the K tiles and the outputs below share LDS

    // merge of the four states: (max, sum) first, then every wavefront's output scaled to the common maximum.
    // Chunks are XOR-swizzled by the row, so that the 16 rows of a store do not meet in a bank.
    const float sum = sum_across_groups(l_total);
    if (kg == 0) {
        m_lds[wave * ROWS + col] = m;
        l_lds[wave * ROWS + col] = sum;
    }
    __syncthreads();
    float top = m_lds[col];
#pragma unroll
    for (int w = 1; w < NW; ++w) top = fmaxf(top, m_lds[w * ROWS + col]);
    const float f = __builtin_amdgcn_exp2f(m - top);
    floatx4 *out = reinterpret_cast<floatx4 *>(o_lds + (wave * ROWS + col) * D);
#pragma unroll
    for (int x = 0; x < VV4; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            floatx4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = total[4 * x + e][i] * f;
            out[(16 * x + 4 * kg + i) ^ col] = y;
        }
    __syncthreads();
    for (int idx = threadIdx.x; idx < ROWS * CHUNKS; idx += NW * 64) {
        const int row = idx / CHUNKS, chunk = idx - row * CHUNKS;
        if (row0 + row >= rows_total) break;             // rows ascend with idx
        float top = m_lds[row];
#pragma unroll
        for (int w = 1; w < NW; ++w) top = fmaxf(top, m_lds[w * ROWS + row]);
        float sum = 0.f;
        floatx4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            sum += l_lds[w * ROWS + row] * __builtin_amdgcn_exp2f(m_lds[w * ROWS + row] - top);
            y += reinterpret_cast<const floatx4 *>(o_lds + (w * ROWS + row) * D)[chunk ^ row];
        }
        const int32_t node = (row0 + row) / G, head = kvh * G + (row0 + row - node * G);
        const int64_t t = int64_t(node_base) + node;
        if (p.splits > 1) {
            const int64_t at = split * p.part_rows + t * p.num_q_heads + head;
            *reinterpret_cast<floatx4 *>(p.part_o + at * D + 4 * chunk) = y;
            if (chunk == 0) *reinterpret_cast<floatx2 *>(p.part_ml + at * 2) = floatx2{top, sum};
            continue;
        }
        y *= sum > 0.f ? 1.f / sum : 0.f;
        *reinterpret_cast<floatx4 *>(p.o + t * p.o_ts + head * p.o_hs + 4 * chunk) = y;
        if (p.lse && chunk == 0)
            p.lse[t * p.num_q_heads + head] = sum > 0.f ? (top + __log2f(sum)) * 0.6931471805599453f : -__builtin_inff();
    }
}

}  // namespace

// Splits of the keys that a small timing model likes best (microseconds, 256 CUs): 4.5 outside the loop and 1.45 (head_dim
// 64: 0.75) per turn of the four wavefronts, in rounds of one work-group per CU, and for splitting the merge kernel: 2.5,
// and per split 0.4 and 0.32 per 1024 rows.  Never fewer than two turns per split.  Measured (us, unsplit -> chosen): 32 heads
// of 64 rows over 1088 keys 30.5 -> 23.7 (3 splits 26.3, 4 23.8, 6 29.9); 8 of 32 over 4128 88 -> 18.4; 4 of 16 over 8016
// 164 -> 22.8; 16 of 64 x 4 sequences, one round unsplit, stays (2 splits 34.5 against 31.8).  The constants are older than
// the kernel's present turn and the present merge: over 700 random shapes that no fit saw what is picked is 0.7 % (head_dim 128) and
// 1.4 % (64) behind the best split count in the geometric mean, 37 % at most.
int attention_f32_splits(const gsd_attn_desc &d, size_t room) {
    const int rows = d.max_nodes * (d.num_q_heads / d.num_kv_heads);
    const int turns = int((int64_t(d.max_prefix) + d.max_nodes + 63) / 64);
    if (d.num_splits > 0) {
        const int forced = d.num_splits < turns ? d.num_splits : turns;
        return forced < 64 ? forced : 64;
    }
    const int cap = turns / 2 < 1 ? 1 : turns / 2 < 64 ? turns / 2 : 64;
    const float tiles = float(d.batch) * float(d.num_kv_heads) * float((rows + 15) / 16);
    const float merge_us = 0.32f / 1024.0f * float(d.total_nodes) * float(d.num_q_heads) * (d.head_dim == 128 ? 1.0f : 0.5f);
    int best = 1;
    float best_us = -1.0f;
    for (int s = 1; s <= cap && attention_workspace(d, s) <= room; ++s) {
        float us = ceilf(tiles * s / 256.0f) * (4.5f + float((turns + s - 1) / s) * (d.head_dim == 128 ? 1.45f : 0.75f));
        if (s > 1) us += 2.5f + (0.4f + merge_us) * s;
        if (best_us < 0.0f || us < best_us) {
            best_us = us;
            best = s;
        }
        if (tiles * s >= 512.0f) break;
    }
    return best;
}

hipError_t launch_attention_f32(const gsd_attn_desc &d, int splits, hipStream_t stream) {
    F32Params p;
    p.q = (const float *)d.q; p.o = (float *)d.o; p.lse = d.lse; p.k = (const float *)d.k; p.v = (const float *)d.v;
    p.kv_offsets = d.kv_offsets; p.prefix_lens = d.prefix_lens; p.node_offsets = d.node_offsets; p.mask = d.mask;
    p.q_ts = d.q_token_stride; p.q_hs = d.q_head_stride; p.o_ts = d.o_token_stride; p.o_hs = d.o_head_stride;
    p.kv_ts = d.kv_token_stride; p.kv_hs = d.kv_head_stride;
    p.groups = d.batch * d.num_kv_heads; p.max_nodes = d.max_nodes; p.num_q_heads = d.num_q_heads;
    p.num_kv_heads = d.num_kv_heads; p.group = d.num_q_heads / d.num_kv_heads; p.words_per_row = d.words_per_row;
    p.scale_log2e = d.softmax_scale * kF32Log2e;
    p.row_tiles = (d.max_nodes * p.group + 15) / 16;
    p.splits = splits;
    p.part_rows = int64_t(d.total_nodes) * d.num_q_heads;
    p.part_o = splits > 1 ? (float *)d.workspace : nullptr;
    p.part_ml = splits > 1 ? p.part_o + splits * p.part_rows * d.head_dim : nullptr;
    const dim3 grid((unsigned)((p.groups + 7) / 8 * 8 * p.row_tiles * splits)), block(kF32Waves * 64);
    const bool near = p.kv_ts < (int64_t(1) << 25);      // 15 rows stay below 2^31 bytes
    if (d.head_dim == 64) {
        if (near) hipLaunchKernelGGL((dag_attention_f32_kernel<64, uint32_t>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((dag_attention_f32_kernel<64, int64_t>), grid, block, 0, stream, p);
    } else {
        if (near) hipLaunchKernelGGL((dag_attention_f32_kernel<128, uint32_t>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((dag_attention_f32_kernel<128, int64_t>), grid, block, 0, stream, p);
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess || splits <= 1) return err;
    AttnParams c = {};                                   // what the merge kernel reads
    c.o = (__bf16 *)d.o; c.lse = d.lse; c.o_ts = d.o_token_stride; c.o_hs = d.o_head_stride;
    c.part_o = p.part_o; c.part_ml = p.part_ml; c.splits = splits;
    c.total_nodes = d.total_nodes; c.num_q_heads = d.num_q_heads;
    return launch_attention_combine(c, d.head_dim, GSD_F32, stream);
}

}  // namespace gsd
