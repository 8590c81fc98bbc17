"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded inputs.
Bit-exact for masks, argmax ids and accepted paths; attention within max-abs 1e-4 (fp32) / 2e-2 (bf16)."""
import numpy as np
import pytest
import torch

from paper_2407_16207_amd.workload import (VerifyConfig, Workload, make_workload, random_dag, f32_to_bf16_bits)

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


@pytest.fixture(scope="module")
def gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import gpu_util
    return gpu_util


_cache = {}


def workload(cfg_id, **kw):
    key = (cfg_id, tuple(sorted(kw.items())))
    if key not in _cache:
        if len(_cache) > 1:          # keep at most two big workloads alive on the host
            _cache.pop(next(iter(_cache)))
        print(f"[gen] config {cfg_id} {kw}", flush=True)
        _cache[key] = make_workload(cfg_id, **kw)
    return _cache[key]


def custom_workload(rng, sizes, prefixes, Hq, Hkv, D, dtype, vocab=97, max_parents=3):
    """Several sequences with general (non-layered) DAGs of different sizes and prefix lengths."""
    B = len(sizes)
    node_offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    offs, pars, e = [np.zeros(1, dtype=np.int32)], [], 0
    for n in sizes:
        o, p = random_dag(rng, n, max_parents)
        offs.append(o[1:] + e)
        pars.append(p)
        e += len(p)
    T = int(node_offsets[-1])
    prefix_lens = np.asarray(prefixes, dtype=np.int32)
    rows = prefix_lens.astype(np.int64) + np.asarray(sizes)
    kv_offsets = np.concatenate([[0], np.cumsum(rows)[:-1]]).astype(np.int64)
    R = int(rows.sum())

    def draw(shape):
        x = rng.standard_normal(shape, dtype=np.float32)
        return x if dtype == "f32" else f32_to_bf16_bits(x)

    cfg = VerifyConfig("custom", B, Hq, Hkv, D, int(min(prefixes)), int(max(prefixes)), 1, max(sizes), max_parents,
                       vocab, 0.5, dtype)
    tokens = rng.integers(0, 6, T).astype(np.int32)                  # tiny token alphabet: ties and long paths
    logits = rng.standard_normal((T, vocab), dtype=np.float32)
    logits[np.arange(T), rng.integers(0, 6, T)] += 6.0
    return Workload(cfg=cfg, seed=0, node_offsets=node_offsets, parent_offsets=np.concatenate(offs).astype(np.int32),
                    parent_idx=np.concatenate(pars).astype(np.int32), tokens=tokens,
                    root_pred=rng.integers(0, 6, B).astype(np.int32), prefix_lens=prefix_lens, kv_offsets=kv_offsets,
                    q=draw((T, Hq, D)), k=draw((R, Hkv, D)), v=draw((R, Hkv, D)),
                    logits=logits if dtype == "f32" else f32_to_bf16_bits(logits),
                    softmax_scale=float(1.0 / np.sqrt(D)))


# ------------------------------------------------------------------------------------------------- mask
@pytest.mark.parametrize("cfg_id", [1, 2, 3, 4, 5])
def test_mask_configs(gpu, ref, cfg_id):
    w = workload(cfg_id, with_qkv=False, with_logits=False)
    d = gpu.DeviceWorkload(w)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = gpu.mask_to_numpy(d.build_mask(flag=flag))
    want, _ = ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)
    assert np.array_equal(got, want)
    assert int(flag.item()) == 0
    if cfg_id == 5:                                   # the same-size tree-shaped comparison mask
        wt = workload(5, with_qkv=False, with_logits=False, tree=True)
        got = gpu.mask_to_numpy(gpu.DeviceWorkload(wt).build_mask())
        assert np.array_equal(got, ref.build_mask(wt.node_offsets, wt.parent_offsets, wt.parent_idx)[0])


def test_mask_general_dags_and_edges(gpu, ref):
    rng = np.random.default_rng(77)
    w = custom_workload(rng, [1, 70, 512, 3, 129, 64, 65], [0] * 7, 1, 1, 64, "f32")
    d = gpu.DeviceWorkload(w)
    got = gpu.mask_to_numpy(d.build_mask())
    assert np.array_equal(got, ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)[0])
    # wider rows than needed: the extra words are zero
    got = gpu.mask_to_numpy(d.build_mask(words_per_row=8))
    want = ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx, words_per_row=8)[0]
    assert np.array_equal(got, want)
    # a deep chain: the longest dependency run the relaxation can meet
    n = 512
    w2 = custom_workload(rng, [n], [0], 1, 1, 64, "f32")
    w2.parent_offsets = np.arange(n + 1, dtype=np.int32)
    w2.parent_idx = np.arange(-1, n - 1, dtype=np.int32)
    got = gpu.mask_to_numpy(gpu.DeviceWorkload(w2).build_mask())
    assert np.array_equal(got, ref.build_mask(w2.node_offsets, w2.parent_offsets, w2.parent_idx)[0])


def test_mask_and_accept_dense_dags(gpu, ref):
    """Nodes with more parents than the kernels keep in registers (4), and a sequence whose parent lists (more than
    6144 entries) do not fit the kernels' LDS copy and are read from memory."""
    for seed, sizes, max_parents in ((5, [40, 200, 512], 9), (6, [512, 300], 40)):
        rng = np.random.default_rng(seed)
        w = custom_workload(rng, sizes, [0] * len(sizes), 1, 1, 64, "f32", vocab=6, max_parents=max_parents)
        per_seq_edges = np.diff(w.parent_offsets[w.node_offsets])
        assert np.diff(w.parent_offsets).max() > 4
        if max_parents == 40:
            assert per_seq_edges.max() > 6144
        d = gpu.DeviceWorkload(w)
        got = gpu.mask_to_numpy(d.build_mask())
        assert np.array_equal(got, ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)[0])
        pred = rng.integers(0, 6, w.total_nodes).astype(np.int32)
        ln, path, bonus, _ = d.accept(logits=False, pred=torch.from_numpy(pred).cuda())
        wl, wp, wb = ref.accept_longest_path(w.node_offsets, w.parent_offsets, w.parent_idx, w.tokens, pred,
                                             w.root_pred)
        assert np.array_equal(ln.cpu().numpy(), wl) and np.array_equal(path.cpu().numpy(), wp)
        assert np.array_equal(bonus.cpu().numpy(), wb)


@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 129, 193, 257, 320, 449, 512])
def test_mask_blocks_of_64(gpu, ref, n):
    """Around the edges of the 64 x 64 blocks: parents within a block, in the one before and far back; no node with more than four
    parents, exactly one (in any lane), and all of them; rows wider than they need to be."""
    rng = np.random.default_rng(n)
    for rep in range(6):
        counts = np.ones(n, dtype=int) if rep < 5 else rng.integers(5, 9, n)
        if 0 < rep < 5:
            counts[:] = rng.integers(1, 5, n)
            counts[n - 1 - rep * 11 % n] = 9
        reach = [n, 3, 64, 70, n, 130][rep]
        offsets, parents = [0], []
        for i in range(n):
            lo = max(0, i - reach)
            pick = rng.choice(i - lo, min(counts[i], i - lo), replace=False) + lo if i else []
            parents += sorted(int(x) for x in pick) or [-1]
            offsets.append(len(parents))
        w = custom_workload(rng, [n], [0], 1, 1, 64, "f32")
        w.parent_offsets, w.parent_idx = np.array(offsets, dtype=np.int32), np.array(parents, dtype=np.int32)
        words = (n + 63) // 64 + (rep % 3) * 5
        got = gpu.mask_to_numpy(gpu.DeviceWorkload(w).build_mask(words_per_row=words))
        assert np.array_equal(got, ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx, words_per_row=words)[0]), rep


@pytest.mark.parametrize("n", [65, 77, 128, 129, 256, 300, 511, 512])
def test_mask_blocks_without_edges_within(gpu, ref, n):
    """Blocks of 64 nodes whose parents all lie in earlier blocks, or are the root, take no steps of their own: no such edge in any
    block, in one block only, one edge in the last lane; with nodes of more than four parents and without."""
    rng = np.random.default_rng(40 + n)
    for rep in range(8):
        deep = int(rng.integers(0, (n + 63) // 64)) if rep % 4 else -1            # the block that has edges within, if any
        offsets, parents = [0], []
        for i in range(n):
            block = i // 64
            few = int(rng.integers(1, 9 if rep >= 4 else 5))
            pick = rng.choice(64 * block, min(few, 64 * block), replace=False).tolist() if block and rep != 4 else []
            if block == deep and i % 64 and (rep % 4 != 3 or i % 64 == 63 or i == n - 1):
                pick.append(int(rng.integers(64 * block, i)))
            parents += sorted(set(pick)) or [-1]
            offsets.append(len(parents))
        w = custom_workload(rng, [n], [0], 1, 1, 64, "f32")
        w.parent_offsets, w.parent_idx = np.array(offsets, dtype=np.int32), np.array(parents, dtype=np.int32)
        got = gpu.mask_to_numpy(gpu.DeviceWorkload(w).build_mask())
        assert np.array_equal(got, ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)[0]), rep


def test_mask_bad_parent_sets_flag(gpu, ref):
    rng = np.random.default_rng(3)
    w = custom_workload(rng, [6], [0], 1, 1, 64, "f32")
    w.parent_offsets = np.array([0, 1, 2, 3, 4, 5, 6], dtype=np.int32)
    w.parent_idx = np.array([-1, 0, 4, 1, 2, -7], dtype=np.int32)     # node 2 names a later node, node 5 garbage
    d = gpu.DeviceWorkload(w)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = gpu.mask_to_numpy(d.build_mask(flag=flag))
    want, want_flag = ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)
    assert int(flag.item()) == 1 == want_flag
    assert np.array_equal(got, want)


# -------------------------------------------------------------------------------------------- attention
def check_attention(gpu, ref, w, d=None, rows=None, **kw):
    d = d or gpu.DeviceWorkload(w)
    mask_ref, _ = ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)
    mask = d.build_mask()
    assert np.array_equal(gpu.mask_to_numpy(mask), mask_ref)
    out, lse = d.attention(mask, return_lse=True, **kw)
    torch.cuda.synchronize()
    got, got_lse = gpu.out_to_f64(out), lse.cpu().numpy().astype(np.float64)
    tol = TOL[w.cfg.dtype]
    if rows is None:
        want, want_lse = ref.dag_attention(w.q, w.k, w.v, w.kv_offsets, w.prefix_lens, w.node_offsets, mask_ref,
                                           w.softmax_scale, return_lse=True)
    else:
        rb, ri, rh = rows
        want, want_lse = ref.dag_attention(w.q, w.k, w.v, w.kv_offsets, w.prefix_lens, w.node_offsets, mask_ref,
                                           w.softmax_scale, rows=rows, return_lse=True)
        t = w.node_offsets[rb] + ri
        got, got_lse = got[t, rh], got_lse[t, rh]
    err = np.abs(got - want).max()
    lse_err = np.abs(got_lse - want_lse).max()
    print(f"[attn] {w.cfg.name} {kw} max-abs err {err:.3e} lse err {lse_err:.3e}", flush=True)
    assert np.isfinite(got).all()
    assert err <= tol, err
    # the bf16 path folds scale*log2(e) into Q (one more bf16 rounding of Q: relative 2^-9 per element, so a few
    # 1e-3 on a score) and sums bf16-rounded probabilities; its log-sum-exp is an auxiliary output
    assert lse_err <= (1e-4 if w.cfg.dtype == "f32" else 1e-2), lse_err
    return out


def planned_kernel(w, **kw):
    """Which kernel the library takes for a bf16 call: 1 or 2 = the one whose wavefronts deal out the keys, with that many row
    groups; 4, 8 or 64 = the other one.  Tests that are about one kernel say which, so that a new fit of the plan cannot empty them."""
    import ctypes

    import paper_2407_16207_amd as gsd
    d = gsd.AttnDesc()
    d.batch, d.total_nodes, d.max_nodes, d.max_prefix = w.cfg.batch, w.total_nodes, w.max_nodes, int(w.prefix_lens.max())
    d.num_q_heads, d.num_kv_heads, d.head_dim, d.dtype = w.cfg.num_q_heads, w.cfg.num_kv_heads, w.cfg.head_dim, gsd.GSD_BF16
    d.words_per_row, d.num_splits, d.softmax_scale = (w.max_nodes + 63) // 64, kw.get("num_splits", 0), w.softmax_scale
    return gsd.load_library().gsd_dag_attention_kernel(ctypes.byref(d))


def test_attention_config1_fp32(gpu, ref):
    check_attention(gpu, ref, workload(1))


@pytest.mark.parametrize("D", [64, 128])
def test_attention_fp32_general(gpu, ref, D):
    rng = np.random.default_rng(10 + D)
    w = custom_workload(rng, [5, 130, 1, 64], [0, 77, 300, 64], 6, 2, D, "f32")
    check_attention(gpu, ref, w)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(1, 1), (3, 1), (16, 2)])
def test_attention_fp32_tile_edges(gpu, ref, D, hq, hkv):
    """Rows and keys one below, at and above the 16-row tile, the 16-key run and the four wavefronts' turn of 64 keys."""
    rng = np.random.default_rng(1000 + D + hq)
    check_attention(gpu, ref, custom_workload(rng, [1, 15, 16, 17, 33, 2], [0, 1, 47, 48, 31, 512], hq, hkv, D, "f32"))


@pytest.mark.parametrize("D", [64, 128])
def test_attention_fp32_all_mask_words(gpu, ref, D):
    """Graphs that reach into every word of a mask row, up to the largest, with prefixes off the grid of 16-key runs: the
    last run of the largest holds one key, and lanes that stand for keys far past the end."""
    rng = np.random.default_rng(1050 + D)
    check_attention(gpu, ref, custom_workload(rng, [512, 512, 501, 193, 449], [17, 2, 63, 32, 5], 3, 1, D, "f32"))


@pytest.mark.parametrize("splits", [0, 2, 3, 64])
@pytest.mark.parametrize("D", [64, 128])
def test_attention_fp32_splits(gpu, ref, D, splits):
    """Splits that end inside the prefix and inside the draft nodes, splits without a key; and a workspace that is missing
    or too small leaves the call unsplit, bit for bit."""
    import paper_2407_16207_amd as gsd
    rng = np.random.default_rng(1100 + D + splits)
    w = custom_workload(rng, [1, 15, 16, 17, 33, 2], [0, 1, 47, 48, 531, 5], 6, 2, D, "f32")
    d = gpu.DeviceWorkload(w)
    out = check_attention(gpu, ref, w, d=d, num_splits=splits)
    mask = d.build_mask()
    alone = d.attention(mask, num_splits=1)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    kept = d.attention(mask, num_splits=splits, workspace=small)
    desc = gsd.make_attn_desc(d.q, d.k, d.v, d.kv_offsets, d.prefix_lens, d.node_offsets, mask, d.max_nodes, d.max_prefix,
                              w.softmax_scale, out=torch.empty_like(d.q), num_splits=splits)
    assert (gsd.gsd_dag_attention_workspace(desc) > 0) == (gsd.gsd_dag_attention_splits(desc) > 1)
    torch.cuda.synchronize()
    assert torch.equal(kept, alone)
    assert (out - alone).abs().max().item() < 1e-5


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n,P,bad", [(40, 37, 3), (40, 37, 39), (16, 0, 0), (33, 64, 32), (300, 90, 150), (20, 30, -5), (70, 500, 69)])
def test_attention_fp32_non_finite_rows_stay_with_those_who_see_them(gpu, D, splits, n, P, bad):
    """A draft node whose K/V row overflowed (or a prefix row, bad < 0) next to keys that are masked: rows that do not see it
    keep every bit of their outputs, rows that do carry its infinities and NaNs in its channels and no others."""
    rng = np.random.default_rng(1200 + D + n + P)
    w = custom_workload(rng, [n, 5], [P, 3], 6, 2, D, "f32")
    row = P + bad
    inf_ch, nan_ch, neg_ch = 1, D // 2 + 3, D - 1
    d = gpu.DeviceWorkload(w)
    mask = d.build_mask()
    want, want_lse = d.attention(mask, num_splits=splits, return_lse=True)
    d.v[row, 1, inf_ch], d.v[row, 1, nan_ch], d.v[row, 1, neg_ch] = np.inf, np.nan, -np.inf
    out, lse = d.attention(mask, num_splits=splits, return_lse=True)
    torch.cuda.synchronize()
    words = gpu.mask_to_numpy(mask)
    sees = np.zeros(w.total_nodes, dtype=bool)
    sees[:n] = True if bad < 0 else (words[:n, bad // 64] >> np.uint64(bad % 64)) & np.uint64(1)
    spoiled = torch.zeros(out.shape, dtype=torch.bool)
    spoiled[torch.from_numpy(sees).nonzero()[:, 0, None, None], torch.arange(3, 6)[:, None], torch.tensor([inf_ch, nan_ch, neg_ch])] = True
    spoiled = spoiled.cuda()
    assert torch.equal(out[~spoiled], want[~spoiled]) and torch.equal(lse, want_lse)
    at = torch.from_numpy(sees).cuda()
    assert (out[at, 3:, inf_ch] == np.inf).all() and out[at, 3:, nan_ch].isnan().all() and (out[at, 3:, neg_ch] == -np.inf).all()
    d.k[row, 1] = np.nan                                     # the scores of the rows that see it, and of nobody else
    d.v[row, 1] = np.nan
    out = d.attention(mask, num_splits=splits)
    assert torch.equal(out[~at], want[~at]) and torch.equal(out[:, :3], want[:, :3]) and out[at, 3:].isnan().all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_split_on_side_streams(gpu, dtype):
    """Split calls on two side streams that bring no workspace, allocations on the current stream in between: each call's
    partials are its own until its merge has read them.  The same bits as calls one after the other."""
    rng = np.random.default_rng(61)
    w = custom_workload(rng, [40, 33], [3000, 2500], 8, 2, 128, dtype)
    d = gpu.DeviceWorkload(w)
    mask = d.build_mask()
    scaled = [d.q, (d.q.float() * 0.5).to(d.q.dtype)]
    want = []
    for q in scaled:
        d.q = q
        want.append(d.attention(mask, num_splits=8))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [[torch.empty_like(d.q) for _ in range(20)] for _ in streams]
    torch.cuda.synchronize()
    for turn in range(20):
        for i, stream in enumerate(streams):
            d.q = scaled[i]
            d.attention(mask, num_splits=8, out=got[i][turn], stream=stream)
            torch.full((8 * w.total_nodes * 8 * 130,), float("nan"), device="cuda")       # the size of the partials
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(x, want[i]) for x in got[i])


@pytest.mark.parametrize("waves", [4, 8, 64])
@pytest.mark.parametrize("splits", [1, 2, 3, 7])
@pytest.mark.parametrize("D", [128, 64])
def test_attention_bf16_small_all_rows(gpu, ref, D, splits, waves):
    """Several row tiles and KV tiles, ragged tails on both axes, GQA, an empty prefix, forced KV splits, both
    work-group shapes (128- and 256-row tiles)."""
    rng = np.random.default_rng(100 + D + splits)
    w = custom_workload(rng, [200, 1, 65, 37], [333, 0, 64, 130], 8, 2, D, "bf16")
    check_attention(gpu, ref, w, num_splits=splits, wg_waves=waves)


@pytest.mark.parametrize("hq,hkv,D", [(2, 2, 128), (2, 2, 64), (6, 2, 128), (6, 2, 64), (16, 2, 128)])
@pytest.mark.parametrize("splits", [0, 3])
def test_attention_bf16_few_rows(gpu, ref, hq, hkv, D, splits):
    """Shapes the library gives to the kernel whose wavefronts deal out the keys: rows and keys one below, at and above its
    32-row groups, 32-key tiles and 128-key steps, more splits than steps, an empty prefix."""
    rng = np.random.default_rng(700 + hq + D + splits)
    w = custom_workload(rng, [1, 5, 10, 11, 21, 32, 33], [0, 1, 31, 117, 107, 96, 300], hq, hkv, D, "bf16")
    assert planned_kernel(w, num_splits=splits) == (2 if (hq, splits) == (16, 3) else 1)
    check_attention(gpu, ref, w, num_splits=splits)


@pytest.mark.parametrize("hq,hkv,D,splits,small,large", [
    (1, 1, 128, 0, 1, 1), (1, 1, 128, 2, 1, 1), (1, 1, 128, 3, 1, 2), (3, 1, 128, 0, 1, 2), (3, 1, 128, 2, 1, None), (3, 1, 128, 3, 2, None),
    (8, 2, 128, 0, 1, 2), (8, 2, 128, 2, 2, None), (4, 2, 128, 2, 1, 2), (5, 1, 64, 0, 1, None), (5, 1, 64, 2, 1, None),
    (3, 1, 64, 0, 1, 1), (2, 1, 64, 2, 1, 1)])
def test_attention_bf16_few_rows_prefixes_of_every_length(gpu, ref, hq, hkv, D, splits, small, large):
    """The prefix ends at every position of a 128-key step, and the graph at the edges of mask words, the last ones among them:
    the words of a tile that reaches into the draft nodes are shifted together from two, ones before the first and nothing behind
    the last.  Few sequences to a call, so that all calls take the kernel that deals out the keys, with `small` row groups for
    graphs of up to 65 nodes and `large` for 449 to 512 (None: those are the other kernel's)."""
    rng = np.random.default_rng(10 * hq + D + splits)
    for part in range(13):                           # prefixes part, part + 13, part + 26 ...
        sizes = [65] + [int(rng.choice([1, 2, 31, 32, 33, 63, 64, 65])) for _ in range(9)]
        w = custom_workload(rng, [sizes[(i + part) % 10] for i in range(10)], list(range(part, 130, 13)), hq, hkv, D, "bf16")
        assert planned_kernel(w, num_splits=splits) == small
        check_attention(gpu, ref, w, num_splits=splits)
    for sizes, prefixes in (([512, 511], [0, 31]), ([481, 480, 449], [32, 127, 128])):
        if large is not None:
            w = custom_workload(rng, sizes, prefixes, hq, hkv, D, "bf16")
            assert planned_kernel(w, num_splits=splits) == large
            check_attention(gpu, ref, w, num_splits=splits)


LONG_CONTEXTS = [          # sizes, prefixes; per (query heads, KV heads, head_dim) the kernel with 0 (chosen), 1 and 3 splits
    ([64, 40, 33], [1500, 900, 2100], {(8, 8, 128): (1, 1, 1), (4, 2, 128): (1, 1, 1), (16, 4, 128): (2, 1, 2), (3, 3, 64): (1, 1, 1),
                                       (8, 2, 64): (1, 1, 1)}),
    ([63, 64, 65, 1], [2500, 1900, 100, 0], {(8, 8, 128): (4, 1, 2), (4, 2, 128): (1, 1, 1), (16, 4, 128): (2, 1, 2),
                                             (3, 3, 64): (1, 1, 1), (8, 2, 64): (1, 1, 1)}),
    ([20, 31, 32], [4000, 3777, 130], {(8, 8, 128): (1, 1, 1), (4, 2, 128): (1, 1, 1), (16, 4, 128): (1, 1, 1), (3, 3, 64): (1, 1, 1),
                                       (8, 2, 64): (1, 1, 1)}),
    ([200, 199, 161], [1000, 871, 0], {(16, 4, 128): (2, 2, None)}), ([150, 97], [2100, 1000], {(16, 2, 128): (None, 2, None)}),
    ([65, 64, 63, 33, 8], [1000, 999, 870, 31, 0], {(16, 2, 128): (2, 2, None)}),
    ([200, 3], [4000, 4001], {(16, 2, 128): (None, 2, None)})]


@pytest.mark.parametrize("sizes,prefixes,heads,splits,kernel", [
    (sizes, prefixes, heads, splits, kernel) for sizes, prefixes, by_heads in LONG_CONTEXTS for heads, kernels in by_heads.items()
    for splits, kernel in zip((0, 1, 3), kernels) if kernel is not None])
def test_attention_bf16_few_rows_long_contexts(gpu, ref, sizes, prefixes, heads, splits, kernel):
    """The same kernel over up to 33 steps: its two buffers come round many times, with rows one below, at and above 32 and 64; at
    head_dim 128 with one row group and with two, unsplit and split."""
    hq, hkv, D = heads
    rng = np.random.default_rng(750 + hq + D + len(sizes))
    w = custom_workload(rng, sizes, prefixes, hq, hkv, D, "bf16")
    assert planned_kernel(w, num_splits=splits) == kernel
    check_attention(gpu, ref, w, num_splits=splits)


def test_attention_bf16_mha_and_odd_group(gpu, ref):
    rng = np.random.default_rng(5)
    check_attention(gpu, ref, custom_workload(rng, [70, 3], [129, 5], 3, 3, 128, "bf16"))     # MHA
    check_attention(gpu, ref, custom_workload(rng, [90, 130], [200, 63], 6, 2, 128, "bf16"))  # group of 3
    check_attention(gpu, ref, custom_workload(rng, [512], [100], 8, 1, 128, "bf16"))          # 4096 rows, 8 words
    check_attention(gpu, ref, custom_workload(rng, [300, 40], [70, 1000], 4, 4, 128, "bf16"), wg_waves=8)


def test_attention_strided_layouts_and_wide_mask_rows(gpu, ref):
    """K/V stored head-major ([Hkv, R, D]) and Q/O with padded rows, reached through the descriptor's strides; mask rows
    wider than the graph needs.  Same numbers as the packed layout, bit for bit."""
    import paper_2407_16207_amd as gsd
    rng = np.random.default_rng(31)
    w = custom_workload(rng, [150, 33], [260, 70], 8, 2, 128, "bf16")
    d = gpu.DeviceWorkload(w)
    mask = d.build_mask(words_per_row=5)
    want = ref.dag_attention(w.q, w.k, w.v, w.kv_offsets, w.prefix_lens, w.node_offsets,
                             ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)[0], w.softmax_scale)
    base = d.attention(mask)
    assert np.abs(gpu.out_to_f64(base) - want).max() <= 2e-2
    k_hm = d.k.permute(1, 0, 2).contiguous().permute(1, 0, 2)          # same values, head-major storage
    v_hm = d.v.permute(1, 0, 2).contiguous().permute(1, 0, 2)
    assert k_hm.stride(1) > k_hm.stride(0)
    q_pad = torch.zeros((d.q.shape[0], d.q.shape[1], 160), dtype=d.q.dtype, device="cuda")[:, :, :128]
    q_pad.copy_(d.q)
    o_pad = torch.zeros_like(q_pad)
    out = gsd.gsd_dag_attention(q_pad, k_hm, v_hm, d.kv_offsets, d.prefix_lens, d.node_offsets, mask, d.max_nodes,
                                d.max_prefix, w.softmax_scale, out=o_pad)
    assert torch.equal(out.contiguous().view(torch.int16), base.view(torch.int16))


@pytest.mark.parametrize("splits", [2, 4, 5, 8, 9, 17, 33])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_merge_of_any_number_of_splits(gpu, ref, dtype, D, splits):
    """Up to and past the outputs that the merge fetches first (4 or 8) and the 16 or 32 lanes of a row; rows over a work-group's end."""
    rng = np.random.default_rng(1200 + D + splits)
    check_attention(gpu, ref, custom_workload(rng, [3, 4], [2300, 40], 3, 3, D, dtype), num_splits=splits)


@pytest.mark.parametrize("splits", [1, 4])
@pytest.mark.parametrize("D", [64, 128])
def test_attention_fp32_strided_layouts(gpu, D, splits):
    """The same for fp32: head-major K/V, Q and O with padded rows, wide mask rows; the bits of the packed layout, and
    nothing written beside O's rows."""
    import paper_2407_16207_amd as gsd
    rng = np.random.default_rng(33 + D)
    w = custom_workload(rng, [150, 33, 1], [260, 70, 9], 8, 2, D, "f32")
    d = gpu.DeviceWorkload(w)
    base, base_lse = d.attention(d.build_mask(), num_splits=splits, return_lse=True)
    k_hm = d.k.permute(1, 0, 2).contiguous().permute(1, 0, 2)
    v_hm = d.v.permute(1, 0, 2).contiguous().permute(1, 0, 2)
    assert k_hm.stride(1) > k_hm.stride(0)
    q_pad = torch.zeros((d.q.shape[0], d.q.shape[1], D + 36), device="cuda")[:, :, :D]
    q_pad.copy_(d.q)
    o_all = torch.full((d.q.shape[0], d.q.shape[1], D + 12), 7.0, device="cuda")
    out, lse = gsd.gsd_dag_attention(q_pad, k_hm, v_hm, d.kv_offsets, d.prefix_lens, d.node_offsets, d.build_mask(words_per_row=5),
                                     d.max_nodes, d.max_prefix, w.softmax_scale, out=o_all[:, :, :D], num_splits=splits,
                                     return_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out, base) and torch.equal(lse, base_lse) and (o_all[:, :, D:] == 7.0).all()


@pytest.mark.parametrize("D", [64, 128])
def test_attention_fp32_rows_far_apart(gpu, D):
    """Row strides up to and beyond 2^25 elements (128 MiB), where offsets within a run of 16 rows no longer fit 32 bits: the
    same bits as with the rows side by side."""
    import paper_2407_16207_amd as gsd
    w = custom_workload(np.random.default_rng(D), [5], [18], 2, 2, D, "f32")
    d = gpu.DeviceWorkload(w)
    mask = d.build_mask()

    def attention(k, v):
        return gsd.gsd_dag_attention(d.q, k, v, d.kv_offsets, d.prefix_lens, d.node_offsets, mask, d.max_nodes, d.max_prefix,
                                     w.softmax_scale)
    want, rows = attention(d.k, d.v), d.k.shape[0]
    for stride in ((1 << 25) - 4, 1 << 25):
        room = torch.empty(rows * stride, dtype=torch.float32, device="cuda")
        k = room.as_strided((rows, 2, D), (stride, D, 1))
        v = room.as_strided((rows, 2, D), (stride, D, 1), 4 * D)
        k.copy_(d.k)
        v.copy_(d.v)
        assert torch.equal(attention(k, v), want), stride
        del room, k, v


def test_attention_chain_equals_causal_sdpa(gpu):
    """A chain-shaped graph is plain causal attention: checked against torch's own SDPA on the GPU in fp32."""
    rng = np.random.default_rng(9)
    n, P, H, D = 150, 100, 4, 128
    w = custom_workload(rng, [n], [P], H, H, D, "bf16")
    w.parent_offsets = np.arange(n + 1, dtype=np.int32)
    w.parent_idx = np.arange(-1, n - 1, dtype=np.int32)
    d = gpu.DeviceWorkload(w)
    out = d.attention(d.build_mask()).float()
    qf = torch.zeros(H, P + n, D, device="cuda")
    qf[:, P:] = d.q.float().permute(1, 0, 2)
    o = torch.nn.functional.scaled_dot_product_attention(qf[None], d.k.float().permute(1, 0, 2)[None],
                                                         d.v.float().permute(1, 0, 2)[None], is_causal=True)[0]
    assert (out - o[:, P:].permute(1, 0, 2)).abs().max().item() <= 2e-2


def sample_rows(w, rng, count, full_seq=None):
    B, N, H = w.cfg.batch, w.cfg.nodes, w.cfg.num_q_heads
    rb, ri, rh = rng.integers(0, B, count), rng.integers(0, N, count), rng.integers(0, H, count)
    if full_seq is not None:
        ii, hh = np.meshgrid(np.arange(N), np.arange(H), indexing="ij")
        rb = np.concatenate([rb, np.full(N * H, full_seq)])
        ri = np.concatenate([ri, ii.ravel()])
        rh = np.concatenate([rh, hh.ravel()])
    return rb.astype(np.int32), ri.astype(np.int32), rh.astype(np.int32)


@pytest.mark.parametrize("cfg_id", [2, 3])
def test_attention_configs_all_rows(gpu, ref, cfg_id):
    check_attention(gpu, ref, workload(cfg_id, with_logits=False))


def test_attention_config4_all_rows(gpu, ref):
    """The headline configuration, in the launch shape the benchmark times: every one of its 2048 x 64 rows against
    the oracle; the same launch again is bit-identical."""
    w = workload(4, with_logits=False)
    d = gpu.DeviceWorkload(w)
    out = check_attention(gpu, ref, w, d=d)
    out2 = d.attention(d.build_mask())
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))


def test_attention_config5_full_size_sampled(gpu, ref):
    """Full-size launch as the benchmark times it; the oracle checks 4096 random (sequence, node, head) rows plus
    every row of one whole sequence (the one with the shortest prefix); then the same-size tree-shaped graph."""
    w = workload(5, with_logits=False)
    rng = np.random.default_rng(5)
    rows = sample_rows(w, rng, 4096, full_seq=int(np.argmin(w.prefix_lens)))
    d = gpu.DeviceWorkload(w)
    out = check_attention(gpu, ref, w, d=d, rows=rows)
    out2 = d.attention(d.build_mask())
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    wt = workload(5, with_logits=False, tree=True)
    wt.q, wt.k, wt.v = w.q, w.k, w.v
    check_attention(gpu, ref, wt, rows=sample_rows(wt, rng, 2048))


# ------------------------------------------------------------------------------------- argmax + acceptance
@pytest.mark.parametrize("cfg_id", [1, 2, 3, 4, 5])
def test_argmax_and_accept_configs(gpu, ref, cfg_id):
    w = workload(cfg_id, with_qkv=False)
    d = gpu.DeviceWorkload(w)
    ln, path, bonus, pred = d.accept()
    torch.cuda.synchronize()
    want_pred = ref.node_argmax(w.logits)
    assert np.array_equal(pred.cpu().numpy(), want_pred)
    wl, wp, wb = ref.accept_longest_path(w.node_offsets, w.parent_offsets, w.parent_idx, w.tokens, want_pred,
                                         w.root_pred)
    assert np.array_equal(ln.cpu().numpy(), wl)
    assert np.array_equal(path.cpu().numpy(), wp)
    assert np.array_equal(bonus.cpu().numpy(), wb)
    print(f"[accept] config {cfg_id} accepted lengths {wl.tolist()[:8]}", flush=True)


def test_argmax_edge_rows(gpu, ref):
    import paper_2407_16207_amd as gsd
    rng = np.random.default_rng(1)
    for vocab in (1, 7, 1000, 32000, 32003):
        x = rng.standard_normal((9, vocab)).astype(np.float32)
        x[0, :] = 0.5                              # a whole row of ties
        x[1, vocab - 1] = 9.0
        x[2, 0] = 9.0
        x[3, :] = -np.inf
        x[4, :] = np.nan
        x[5, ::3] = np.nan
        if vocab > 10:
            x[6, [vocab - 2, 5, vocab // 2]] = 7.0
        got = gsd.gsd_node_argmax(torch.from_numpy(x).cuda()).cpu().numpy()
        assert np.array_equal(got, ref.node_argmax(x)), vocab
        xb = f32_to_bf16_bits(x)                   # NaN and -inf survive the rounding
        got = gsd.gsd_node_argmax(gpu.to_dev(xb)).cpu().numpy()
        assert np.array_equal(got, ref.node_argmax(xb)), vocab
    # rows that start off the 16-byte grid (odd row stride)
    big = torch.from_numpy(rng.standard_normal((5, 1003)).astype(np.float32)).cuda()
    view = big[:, 1:1000]
    got = gsd.gsd_node_argmax(view).cpu().numpy()
    assert np.array_equal(got, np.argmax(view.cpu().numpy(), axis=1))


def test_accept_general_dags_with_ties(gpu, ref):
    rng = np.random.default_rng(2024)
    for trial in range(6):
        sizes = [int(x) for x in rng.integers(1, 200, 5)] + [512, 1]
        w = custom_workload(rng, sizes, [0] * len(sizes), 1, 1, 64, "f32", vocab=6, max_parents=4)
        d = gpu.DeviceWorkload(w)
        pred = rng.integers(0, 6, w.total_nodes).astype(np.int32)
        ln, path, bonus, _ = d.accept(logits=False, pred=torch.from_numpy(pred).cuda())
        wl, wp, wb = ref.accept_longest_path(w.node_offsets, w.parent_offsets, w.parent_idx, w.tokens, pred,
                                             w.root_pred)
        assert np.array_equal(ln.cpu().numpy(), wl) and np.array_equal(path.cpu().numpy(), wp)
        assert np.array_equal(bonus.cpu().numpy(), wb)
        assert wl.max() > 1


@pytest.mark.parametrize("parents", [4, 5, 12, 13, 30])
@pytest.mark.parametrize("n", [64, 65, 129, 257, 512])
def test_accept_parent_counts(gpu, ref, n, parents):
    """Up to four parents of a node are kept in registers, the accepted ones of the others in LDS, fetched eight at a time; at 512
    nodes of 30 parents the lists go past the LDS room of 6144 entries part of the way."""
    rng = np.random.default_rng(n + parents)
    w = custom_workload(rng, [n, n], [0, 0], 1, 1, 64, "f32", vocab=6)
    off, par = [0], []
    for seq in range(2):
        for i in range(n):
            k = min(i + 1, parents if seq == 0 or i % 3 else min(parents, 7))
            par += sorted(rng.choice(np.arange(-1, i), size=k, replace=False).tolist())
            off.append(len(par))
    w.parent_offsets, w.parent_idx = np.asarray(off, dtype=np.int32), np.asarray(par, dtype=np.int32)
    w.tokens = rng.integers(0, 3, 2 * n).astype(np.int32)
    pred, w.root_pred = rng.integers(0, 3, 2 * n).astype(np.int32), rng.integers(0, 3, 2).astype(np.int32)
    ln, path, bonus, _ = gpu.DeviceWorkload(w).accept(logits=False, pred=torch.from_numpy(pred).cuda())
    wl, wp, wb = ref.accept_longest_path(w.node_offsets, w.parent_offsets, w.parent_idx, w.tokens, pred, w.root_pred)
    assert np.array_equal(ln.cpu().numpy(), wl) and np.array_equal(path.cpu().numpy(), wp)
    assert np.array_equal(bonus.cpu().numpy(), wb)


def test_end_to_end_verify_step_config2(gpu, ref):
    """All three ABI calls back to back on one stream, as one verify step."""
    w = workload(2)
    d = gpu.DeviceWorkload(w)
    mask = d.build_mask()
    out = d.attention(mask)
    ln, path, bonus, pred = d.accept()
    torch.cuda.synchronize()
    mask_ref, _ = ref.build_mask(w.node_offsets, w.parent_offsets, w.parent_idx)
    want = ref.dag_attention(w.q, w.k, w.v, w.kv_offsets, w.prefix_lens, w.node_offsets, mask_ref, w.softmax_scale)
    assert np.abs(gpu.out_to_f64(out) - want).max() <= 2e-2
    wl, wp, wb = ref.accept_longest_path(w.node_offsets, w.parent_offsets, w.parent_idx, w.tokens,
                                         ref.node_argmax(w.logits), w.root_pred)
    assert np.array_equal(ln.cpu().numpy(), wl) and np.array_equal(path.cpu().numpy(), wp)
    assert np.array_equal(bonus.cpu().numpy(), wb)
