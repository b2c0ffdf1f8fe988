"""GPU parity: every C-ABI call, and the whole iteration, against the CPU oracle on the same seeded inputs.

Bars: bit-exact for flags, index lists, counts, pruned row ends, gathered rows and cache state;
REL_TOL_F32 for aggregation and linear outputs (relative error as defined in helpers.rel_err_rows).
"""
import os

import numpy as np
import pytest

from fg_inputs import features, workload as wl
from oracle import freshgnn_oracle as O
from tests import helpers as T
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

REL_TOL_F32 = 1e-5


def random_seeds(default):
    """Seeds of the random-configuration tests: FG_RANDOM_SEEDS of them (default given per test), starting at
    FG_RANDOM_SEED_BASE (default 0), so that a longer run can cover seeds that the default run does not."""
    base = int(os.environ.get("FG_RANDOM_SEED_BASE", "0"))
    return range(base, base + int(os.environ.get("FG_RANDOM_SEEDS", str(default))))


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2301_07482_amd import binding as B
    assert torch.cuda.is_available()
    return torch, B


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# ------------------------------------------------------------------------------------------------ fg_gather

@pytest.mark.parametrize("row_bytes,dtype", [(256, np.float32), (400, np.float32), (512, np.float32), (1024, np.float32),
                                             (1536, np.float16), (2048, np.float16), (24, np.float32), (6, np.float16)])
def test_gather_bit_exact(env, row_bytes, dtype):
    torch, B = env
    r = np.random.default_rng(row_bytes)
    elems = row_bytes // np.dtype(dtype).itemsize
    table_rows, n_dst, max_count = 5000, 3000, 2500
    table = r.standard_normal((table_rows, elems)).astype(dtype)
    for count, use_pos in [(max_count, True), (1733, True), (1, False), (0, True), (1733, False)]:
        src = r.integers(0, table_rows, max_count).astype(np.int32)
        pos = r.permutation(n_dst)[:max_count].astype(np.int32)
        dst0 = r.standard_normal((n_dst, elems)).astype(dtype)
        t_tab, t_src, t_pos, t_dst = dev(torch, table), dev(torch, src), dev(torch, pos), dev(torch, dst0)
        t_cnt = torch.tensor([count], dtype=torch.int64, device="cuda")
        B.fg_gather(t_tab, table_rows, row_bytes, row_bytes, t_src, t_pos if use_pos else None, t_cnt, max_count, t_dst,
                    n_dst, row_bytes, 0, torch.cuda.current_stream().cuda_stream)
        want = dst0.copy()
        O.gather(lambda idx: table[idx], src[:count], want, pos[:count] if use_pos else None)
        got = t_dst.cpu().numpy()
        assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), (row_bytes, count, use_pos)


def test_gather_skips_out_of_range_and_strided_rows(env):
    torch, B = env
    r = np.random.default_rng(0)
    table = r.standard_normal((100, 40)).astype(np.float32)        # 32 floats copied out of rows of 40
    src = np.array([5, -1, 100, 7, 99, 0], dtype=np.int32)
    pos = np.array([0, 1, 2, 50, 3, -4], dtype=np.int32)
    dst0 = np.zeros((10, 36), dtype=np.float32)
    t_dst = dev(torch, dst0)
    B.fg_gather(dev(torch, table), 100, 160, 128, dev(torch, src), dev(torch, pos), None, 6, t_dst, 10, 144, 0, None)
    want = dst0.copy()
    want[0, :32] = table[5, :32]
    want[3, :32] = table[99, :32]
    assert np.array_equal(t_dst.cpu().numpy(), want)


# ------------------------------------------------------------------------------------------------ fg_lookup_prune

def _random_block(r, n, n_src, max_deg):
    deg = r.integers(0, max_deg + 1, n)
    gap = r.integers(0, 2, n)                                    # unused col entries between rows are allowed
    start = np.cumsum(np.concatenate([[0], (deg + gap)[:-1]])).astype(np.int32)
    end = (start + deg).astype(np.int32)
    nnz = int(end[-1] + gap[-1]) if n else 0
    col = r.integers(0, n_src, max(nnz, 1)).astype(np.int32)
    return start, end, col, nnz


@pytest.mark.parametrize("n,n_src,max_deg,seed", [(1, 5, 3, 0), (1000, 4000, 6, 1), (1024, 1024, 0, 2), (5000, 30000, 25, 3),
                                                   (70001, 200000, 4, 4)])
def test_lookup_prune_matches_oracle(env, n, n_src, max_deg, seed):
    torch, B = env
    r = np.random.default_rng(seed)
    N, cap, t_stale, it = 300000, 4096, 5, 9
    ids = r.permutation(N)[:n].astype(np.int32)
    live = (r.random(n) < 0.7)
    start, end, col, nnz = _random_block(r, n, n_src, max_deg)
    # a cache state with valid, stale, recycled and checked-out entries: the same updates on both sides
    oc = O.HistoricalCache(N, cap, 4, t_stale)
    cache = B.fg_cache_create(N, [cap], [4], B.FG_F32, t_stale, None)
    try:
        for a in range(2, 9):
            sub = r.permutation(n)[:min(n, 900)]
            ids_a = np.concatenate([ids[sub], r.permutation(N)[:300].astype(np.int32)])
            ids_a = ids_a[np.sort(np.unique(ids_a, return_index=True)[1])]
            gn_a = np.exp(r.standard_normal(len(ids_a))).astype(np.float32)
            rows_a = np.zeros((len(ids_a), 4), np.float32)
            look = O.lookup_prune(oc, a, ids_a, None, None, None, None, 0)
            O.cache_update(oc, a, ids_a, None, look["hit"], gn_a, 0.6, rows_a)
            hit_dev, _, _ = _device_update(torch, B, cache, a, ids_a, None, gn_a, 0.6, rows_a)
            assert np.array_equal(hit_dev, look["hit"])
        for use_cache, use_live in [(True, True), (True, False), (False, True)]:
            want_end = end.copy()
            want = O.lookup_prune(oc if use_cache else None, it, ids, live if use_live else None, start, want_end, col, n_src)
            t_end = dev(torch, end)
            t_live_src = torch.full((n_src,), 7, dtype=torch.uint8, device="cuda")
            t_hit = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
            t_hp, t_hs, t_np, t_ni = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(4))
            t_cnt = torch.zeros(3, dtype=torch.int64, device="cuda")
            wsb = B.fg_workspace_bytes(B.FG_WS_LOOKUP_PRUNE, n)
            ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
            B.fg_lookup_prune(cache if use_cache else None, 1, it, dev(torch, ids), n,
                              dev(torch, live.astype(np.uint8)) if use_live else None, dev(torch, start), t_end,
                              dev(torch, col), nnz, n_src, t_live_src, t_hit, t_hp, t_hs, t_np, t_ni, t_cnt, ws, wsb, None)
            cnt = t_cnt.cpu().numpy()
            assert tuple(cnt) == want["counts"]
            assert np.array_equal(t_hit.cpu().numpy().astype(bool), want["hit"])
            assert np.array_equal(t_hp.cpu().numpy()[:cnt[1]], want["hit_pos"])
            assert np.array_equal(t_hs.cpu().numpy()[:cnt[1]], want["hit_slot"])
            assert np.array_equal(t_np.cpu().numpy()[:cnt[2]], want["normal_pos"])
            assert np.array_equal(t_ni.cpu().numpy()[:cnt[2]], ids[want["normal_pos"]])
            assert np.array_equal(t_end.cpu().numpy(), want_end)
            assert np.array_equal(t_live_src.cpu().numpy().astype(bool), want["live_src"])
            if use_cache and n >= 1000:
                assert cnt[1] > 0
            # the same layer through fg_top_down as a list of one layer: with the size as a host integer, and with the arrays
            # padded by garbage (ids that may be cached, live flags set, row ranges out of range) behind a count in device memory
            pad = 1500
            for counted in (False, True):
                m = n + pad if counted else n
                g_ids = np.concatenate([ids, r.permutation(N)[:m - n].astype(np.int32)])
                g_live = np.concatenate([live if use_live else np.ones(n, bool), np.ones(m - n, bool)]).astype(np.uint8)
                g_start = np.concatenate([start, r.integers(-5, nnz + 5, m - n).astype(np.int32)])
                g_end = np.concatenate([end, r.integers(-5, nnz + 5, m - n).astype(np.int32)])
                t_end = dev(torch, g_end)
                ns = max(n_src, m)      # the layer below is bounded like this one
                t_live_src = torch.full((ns,), 7, dtype=torch.uint8, device="cuda")
                t_hit = torch.full((m,), 9, dtype=torch.uint8, device="cuda")
                t_hp, t_hs, t_np, t_ni = (torch.full((m,), -7, dtype=torch.int32, device="cuda") for _ in range(4))
                t_cnt = torch.zeros(3, dtype=torch.int64, device="cuda")
                t_n = dev(torch, np.asarray([n], dtype=np.int64))
                # (the descriptors hold addresses only: the tensors must outlive the calls)
                t_ids, t_glive, t_start, t_col = dev(torch, g_ids), dev(torch, g_live), dev(torch, g_start), dev(torch, col)
                layers = B.top_down_layers([dict(cache_layer=1 if use_cache else 0, ids_dev=t_ids, n=m,
                                                 live_dev=t_glive if (use_live or counted) else None,
                                                 row_start_dev=t_start, row_end_dev=t_end, col_dev=t_col, nnz=nnz,
                                                 n_src=ns, live_src_dev=t_live_src, hit_dev=t_hit, hit_pos_dev=t_hp, hit_slot_dev=t_hs,
                                                 normal_pos_dev=t_np, normal_ids_dev=t_ni, counts_dev=t_cnt,
                                                 n_dev=t_n if counted else None)])
                wsb2 = B.fg_top_down_workspace_bytes(layers)
                ws2 = torch.zeros(wsb2, dtype=torch.uint8, device="cuda")
                for _ in range(2):      # twice into the same workspace: every call must leave its marks cleared
                    t_end.copy_(dev(torch, g_end))
                    B.fg_top_down(cache if use_cache else None, it, layers, ws2, wsb2, None)
                cnt = t_cnt.cpu().numpy()
                assert tuple(cnt) == want["counts"], f"fg_top_down, counted={counted}"
                assert np.array_equal(t_hit.cpu().numpy()[:n].astype(bool), want["hit"]) and not t_hit[n:].any().item()
                assert np.array_equal(t_hp.cpu().numpy()[:cnt[1]], want["hit_pos"])
                assert np.array_equal(t_hs.cpu().numpy()[:cnt[1]], want["hit_slot"])
                assert np.array_equal(t_np.cpu().numpy()[:cnt[2]], want["normal_pos"])
                assert np.array_equal(t_ni.cpu().numpy()[:cnt[2]], ids[want["normal_pos"]])
                assert np.array_equal(t_end.cpu().numpy()[:n], want_end) and np.array_equal(t_end.cpu().numpy()[n:], g_end[n:])
                assert np.array_equal(t_live_src.cpu().numpy()[:n_src].astype(bool), want["live_src"]) and not t_live_src[n_src:].any().item()
                assert not ws2[(wsb2 // 2 + 255) // 256 * 256:].any().item(), "the marks must be all zero between calls"
    finally:
        B.fg_cache_destroy(cache)


def test_top_down_clears_liveness_of_the_smallest_batches(env):
    """One seed with two neighbours, no cache, then one seed without neighbours into the same buffers: the second pass
    must not see the first one's liveness marks (a layer below with fewer than four positions is cleared too)."""
    torch, B = env
    z = lambda n, dt: torch.zeros(max(n, 1), dtype=dt, device="cuda")
    live0, hit1, hit0 = torch.full((3,), 5, dtype=torch.uint8, device="cuda"), z(1, torch.uint8), z(3, torch.uint8)
    lists = {l: [z(n, torch.int32) for _ in range(4)] for l, n in ((1, 1), (0, 3))}
    counts = torch.zeros((2, 3), dtype=torch.int64, device="cuda")
    ids1, ids0 = dev(torch, np.array([7], np.int32)), dev(torch, np.array([7, 3, 9], np.int32))
    start, col = dev(torch, np.array([0], np.int32)), dev(torch, np.array([1, 2], np.int32))
    for end_host, want_live in (([2], [1, 1, 1]), ([0], [1, 0, 0])):
        end = dev(torch, np.array(end_host, np.int32))
        specs = [dict(cache_layer=0, ids_dev=ids1, n=1, live_dev=None, row_start_dev=start, row_end_dev=end, col_dev=col, nnz=2,
                      n_src=3, live_src_dev=live0, hit_dev=hit1, hit_pos_dev=lists[1][0], hit_slot_dev=lists[1][1],
                      normal_pos_dev=lists[1][2], normal_ids_dev=None, counts_dev=counts.data_ptr() + 24),
                 dict(cache_layer=0, ids_dev=ids0, n=3, live_dev=live0, row_start_dev=None, row_end_dev=None, col_dev=None, nnz=0,
                      n_src=0, live_src_dev=None, hit_dev=hit0, hit_pos_dev=lists[0][0], hit_slot_dev=lists[0][1],
                      normal_pos_dev=lists[0][2], normal_ids_dev=lists[0][3], counts_dev=counts.data_ptr())]
        layers = B.top_down_layers(specs)
        wsb = B.fg_top_down_workspace_bytes(layers)
        ws = torch.zeros(wsb + 16, dtype=torch.uint8, device="cuda")
        B.fg_top_down(None, 0, layers, ws, wsb, None)
        torch.cuda.synchronize()
        assert live0.cpu().numpy().tolist() == want_live
        n_in = int(counts[0, 2].item())
        assert n_in == sum(want_live) and lists[0][2][:n_in].cpu().numpy().tolist() == [j for j in range(3) if want_live[j]]
        assert lists[0][3][:n_in].cpu().numpy().tolist() == [[7, 3, 9][j] for j in range(3) if want_live[j]]


@pytest.mark.parametrize("n", [1025, 30_001, 262_144])
def test_top_down_whose_chunks_give_up_counts_nothing(env, n):
    """Waits of one to three polls: a layer's lists are those of patient chunks, or all its counts say that some gave up. The pass behind it, in the
    same workspace, is whole again."""
    torch, B = env
    r = np.random.default_rng(n)
    live = r.random(n) < 0.6
    want = np.flatnonzero(live)
    t_live, ids = dev(torch, live.astype(np.uint8)), dev(torch, r.permutation(n).astype(np.int32))
    hit = torch.zeros(n, dtype=torch.uint8, device="cuda")
    lists = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(4)]
    cnt = torch.zeros(3, dtype=torch.int64, device="cuda")
    layers = B.top_down_layers([dict(cache_layer=0, ids_dev=ids, n=n, live_dev=t_live, hit_dev=hit, hit_pos_dev=lists[0], hit_slot_dev=lists[1],
                                     normal_pos_dev=lists[2], normal_ids_dev=lists[3], counts_dev=cnt)])
    wsb = B.fg_top_down_workspace_bytes(layers)
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    gave_up = 0
    try:
        for polls in [1, 2, 3, 0] * 5:
            lists[2].fill_(-9)
            B.fg_set_tuning("wait_polls", polls)
            B.fg_top_down(None, 0, layers, ws, wsb, None)
            counts = cnt.tolist()
            if counts == [-1] * 3 and polls:
                gave_up += 1
                continue
            assert counts == [len(want), 0, len(want)]
            assert np.array_equal(lists[2].cpu().numpy()[:len(want)], want) and torch.equal(lists[3][:len(want)], ids[lists[2][:len(want)].long()])
    finally:
        B.fg_set_tuning("wait_polls", 0)
    print(f"{gave_up} of 15 gave up")


def _device_update(torch, B, cache, i, ids, live, gn, p, rows, misalign=False, two_parts=False):
    """Lookup (no block) followed by the update on the device; returns the hit flags. `misalign` puts the norms
    and the liveness flags at addresses that are not multiples of 16 and 4 bytes."""
    n = len(ids)
    wsb = max(B.fg_workspace_bytes(B.FG_WS_LOOKUP_PRUNE, n), B.fg_workspace_bytes(B.FG_WS_CACHE_UPDATE, n))
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    t_ids = dev(torch, ids)
    t_live = None if live is None else dev(torch, live.astype(np.uint8))
    t_gn = dev(torch, gn)
    if misalign:
        t_gn = torch.cat([t_gn[:1], t_gn])[1:]
        t_live = None if t_live is None else torch.cat([t_live[:1], t_live])[1:]
        assert n == 0 or t_gn.data_ptr() % 16 != 0
    t_hit = torch.zeros(max(n, 1), dtype=torch.uint8, device="cuda")
    t_l = [torch.zeros(max(n, 1), dtype=torch.int32, device="cuda") for _ in range(3)]
    t_cnt = torch.zeros(3, dtype=torch.int64, device="cuda")
    B.fg_lookup_prune(cache, 1, i, t_ids, n, t_live, None, None, None, 0, 0, None, t_hit, t_l[0], t_l[1], t_l[2], None,
                      t_cnt, ws, wsb, None)
    t_stats = torch.zeros(4, dtype=torch.int64, device="cuda")
    t_rows = dev(torch, rows)
    if two_parts:
        specs = B.update_layers([dict(layer=1, n=n, ids_dev=t_ids, live_dev=t_live, hit_dev=t_hit, gnorm_dev=t_gn, h_dev=t_rows,
                                      h_stride=rows.shape[1] * 4, stats_dev=t_stats)])
        B.fg_cache_update_select(cache, i, p, specs, ws, wsb, None)
        B.fg_cache_update_commit(cache, i, specs, ws, wsb, None)
    else:
        B.fg_cache_update(cache, 1, i, t_ids, n, t_live, t_hit, t_gn, p, t_rows, rows.shape[1] * 4, t_stats, ws, wsb, None)
    return t_hit.cpu().numpy()[:n].astype(bool), t_l[1].cpu().numpy(), t_stats.cpu().numpy().tolist()


# ------------------------------------------------------------------------------------------------ fg_aggregate

@pytest.mark.parametrize("dim,dtype,max_deg,n", [(64, "f32", 10, 700), (100, "f32", 15, 3000), (128, "f32", 15, 5000),
                                                 (256, "f32", 10, 900), (128, "f32", 150, 300), (768, "f16", 25, 400),
                                                 (1024, "bf16", 15, 300), (4, "f32", 3, 50),
                                                 (320, "f32", 12, 500), (544, "f32", 8, 300)])   # 80 and 136 pieces: 32-lane groups
def test_aggregate_matches_oracle(env, dim, dtype, max_deg, n):
    torch, B = env
    r = np.random.default_rng(dim + max_deg)
    n_src = 4 * n
    start, end, col, nnz = _random_block(r, n, n_src, max_deg)
    rows = np.sort(r.permutation(n)[: int(0.8 * n)]).astype(np.int32)
    h64 = r.standard_normal((n_src, dim))
    code = {"f32": B.FG_F32, "f16": B.FG_F16, "bf16": B.FG_BF16}[dtype]
    tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    h = O.round_to(h64, dtype)
    t_h = torch.from_numpy(h.astype(np.float32)).cuda().to(tdt) if dtype == "bf16" else dev(torch, h)
    esz = 2 if dtype != "f32" else 4
    for out_dtype in (["f32"] if dtype == "f32" else ["f32", "bf16"]):
        ocode = {"f32": B.FG_F32, "bf16": B.FG_BF16}[out_dtype]
        otd = {"f32": torch.float32, "bf16": torch.bfloat16}[out_dtype]
        t_out = torch.full((len(rows) + 3, dim), 5.0, dtype=otd, device="cuda")
        t_cnt = torch.tensor([len(rows)], dtype=torch.int64, device="cuda")
        B.fg_aggregate(dev(torch, start), dev(torch, end), dev(torch, col), nnz, n, dev(torch, rows), t_cnt, len(rows) + 3,
                       t_h, n_src, dim * esz, dim, code, t_out, dim * (4 if out_dtype == "f32" else 2), ocode, None)
        want = O.round_to(O.aggregate(start, end, col, rows, h), out_dtype).astype(np.float32)
        got = G.to_f32(t_out)
        assert np.all(got[len(rows):] == 5.0)                       # rows past the device-side count are untouched
        tol = REL_TOL_F32 if out_dtype == "f32" else 2e-2
        assert T.rel_err_rows(got[:len(rows)], want) <= tol
        # fp64 accumulation and one rounding: in fact (almost) every element is the correctly rounded mean
        assert (got[:len(rows)] == want).mean() > 0.999
        empty = (end[rows] == start[rows])
        assert empty.any() and np.all(got[:len(rows)][empty] == 0)


@pytest.mark.parametrize("dim,dtype,max_deg,n", [(128, "f32", 15, 3000), (100, "f32", 70, 500), (768, "f16", 25, 300),
                                                 (320, "f32", 12, 400)])
def test_gather_aggregate_equals_gather_then_aggregate(env, dim, dtype, max_deg, n):
    torch, B = env
    r = np.random.default_rng(dim + n)
    n_src, table_rows = 4 * n, 50000
    start, end, col, nnz = _random_block(r, n, n_src, max_deg)
    rows = np.sort(r.permutation(n)[: int(0.7 * n)]).astype(np.int32)
    src_ids = r.permutation(table_rows)[:n_src].astype(np.int32)
    code = {"f32": B.FG_F32, "f16": B.FG_F16}[dtype]
    esz = 4 if dtype == "f32" else 2
    table = O.round_to(r.standard_normal((table_rows, dim)), dtype)
    out_dtype = "f32" if dtype == "f32" else "bf16"
    ocode = {"f32": B.FG_F32, "bf16": B.FG_BF16}[out_dtype]
    t_out = torch.zeros((len(rows), dim), dtype={"f32": torch.float32, "bf16": torch.bfloat16}[out_dtype], device="cuda")
    t_cnt = torch.tensor([len(rows)], dtype=torch.int64, device="cuda")
    t_self = torch.zeros((n_src, dim), dtype=torch.float32 if dtype == "f32" else torch.float16, device="cuda")
    B.fg_gather_aggregate(dev(torch, start), dev(torch, end), dev(torch, col), nnz, n, dev(torch, rows), t_cnt, len(rows),
                          dev(torch, src_ids), n_src, dev(torch, table), table_rows, dim * esz, dim, code, t_out,
                          dim * (4 if out_dtype == "f32" else 2), ocode, t_self, dim * esz, n_src, None)
    # the listed rows' own features are copied bit for bit, nothing else is written
    want_self = np.zeros((n_src, dim), dtype=table.dtype)
    want_self[rows] = table[src_ids[rows]]
    assert np.array_equal(t_self.cpu().numpy().view(np.uint8), want_self.view(np.uint8))
    # oracle: gather the input rows, then aggregate
    h0 = np.zeros((n_src, dim), dtype=table.dtype)
    O.gather(lambda idx: table[idx], src_ids, h0, None)
    want = O.round_to(O.aggregate(start, end, col, rows, h0), out_dtype).astype(np.float32)
    got = G.to_f32(t_out)
    assert T.rel_err_rows(got, want) <= (REL_TOL_F32 if out_dtype == "f32" else 2e-2)
    assert (got == want).mean() > 0.999


# ------------------------------------------------------------------------------------------------ fg_linear

def _linear_case(torch, B, r, n_src, n_rows, max_rows, d_in, d_out, relu, W=None, bias=None):
    h = r.standard_normal((n_src, d_in)).astype(np.float32)
    agg = r.standard_normal((max_rows, d_in)).astype(np.float32) * 0.3
    rows = np.sort(r.permutation(n_src)[:max_rows]).astype(np.int32)
    if W is None:
        W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    if bias is None:
        bias = (0.1 * r.standard_normal(d_out)).astype(np.float32)
    t_out = torch.full((n_src, d_out), -3.0, dtype=torch.float32, device="cuda")
    t_cnt = torch.tensor([n_rows], dtype=torch.int64, device="cuda")
    B.fg_linear(dev(torch, h), n_src, d_in * 4, B.FG_F32, dev(torch, agg), d_in * 4, dev(torch, rows), t_cnt, max_rows, d_in,
                d_out, dev(torch, W), B.FG_F32, dev(torch, bias), 1 if relu else 0, t_out, n_src, d_out * 4, B.FG_F32, None)
    got = t_out.cpu().numpy()
    want = O.round_to(O.linear(h[rows[:n_rows]], agg[:n_rows], W, bias, relu), "f32")
    untouched = np.ones(n_src, bool)
    untouched[rows[:n_rows]] = False
    assert np.all(got[untouched] == -3.0)
    return got[rows[:n_rows]], want, h[rows[:n_rows]], agg[:n_rows]


def test_linear_identity_panels_pin_operand_layout(env):
    """W = [I;0] returns the node's own rows, W = [0;I] the neighbour means: exact in any accumulation order,
    and wrong for any mistake in the matrix-core operand or accumulator layout."""
    torch, B = env
    r = np.random.default_rng(0)
    for d, variant in ((64, 0), (128, 0), (100, 0), (64, 8), (128, 32), (96, 8), (128, 301), (64, 302)):
        B.fg_set_tuning("linear_tile", variant)
        I, Z = np.eye(d, dtype=np.float32), np.zeros((d, d), np.float32)
        zero = np.zeros(d, np.float32)
        got, want, hs, ag = _linear_case(torch, B, r, 700, 333, 400, d, d, False, np.vstack([I, Z]), zero)
        assert np.array_equal(got, hs)
        got, want, hs, ag = _linear_case(torch, B, r, 700, 333, 400, d, d, False, np.vstack([Z, I]), zero)
        assert np.array_equal(got, ag)
        perm = r.permutation(d)
        got, want, hs, ag = _linear_case(torch, B, r, 700, 333, 400, d, d, True, np.vstack([I[perm], Z]), zero)
        assert np.array_equal(got, np.maximum(hs[:, np.argsort(perm)], 0))
    B.fg_set_tuning("linear_tile", 0)


@pytest.mark.parametrize("d_in,d_out,n_rows,max_rows,relu", [(64, 64, 1000, 1200, True), (100, 256, 777, 777, True),
                                                             (128, 256, 4097, 5000, True), (256, 256, 129, 200, False),
                                                             (256, 256, 1, 128, True), (64, 64, 0, 128, True),
                                                             (4, 4, 130, 130, False), (128, 260, 300, 300, True),
                                                             (96, 96, 500, 600, True), (160, 72, 900, 900, False),
                                                             (128, 256, 20000, 20000, True)])
@pytest.mark.parametrize("variant", [0, 8, 32, 64, 301, 302])
def test_linear_matches_oracle(env, d_in, d_out, n_rows, max_rows, relu, variant):
    """variant: the fp32 kernel forced through the tuning key (0 = the library's own choice by problem size; a
    variant that does not support the shape falls back to the LDS-tiled kernel)."""
    torch, B = env
    r = np.random.default_rng(d_in * 7 + d_out)
    B.fg_set_tuning("linear_tile", variant)
    try:
        got, want, _, _ = _linear_case(torch, B, r, max_rows + 500, n_rows, max_rows, d_in, d_out, relu)
    finally:
        B.fg_set_tuning("linear_tile", 0)
    assert got.shape == want.shape
    err = T.rel_err_rows(got, want)
    print(f"linear {d_in}x{d_out} rows {n_rows} variant {variant}: rel err {err:.3e}")
    assert err <= REL_TOL_F32


@pytest.mark.parametrize("max_rows", [1, 1024, 1025])      # 9 column panels: up to 1024 rows a workgroup per 32 x 32 results
@pytest.mark.parametrize("d_in", [4, 28, 36, 132, 224, 228, 252, 260])
def test_linear_of_few_rows_of_any_width(env, d_in, max_rows):
    """Widths around multiples of 32 whose K is shared out between the wavefronts of a workgroup (one or two chunks each, some none), the
    widest that is and the next, on both sides of the number of rows up to which they are."""
    torch, B = env
    got, want, _, _ = _linear_case(torch, B, np.random.default_rng(d_in), max_rows + 50, max(1, max_rows - 7), max_rows, d_in, 260, False)
    assert T.rel_err_rows(got, want) <= REL_TOL_F32


@pytest.mark.parametrize("variant", [0, 301, 302, 32, 64])
@pytest.mark.parametrize("d_in,d_out", [(100, 256), (36, 64), (4, 32), (28, 96)])
def test_linear_width_not_a_multiple_of_32_ignores_what_follows_a_row(env, d_in, d_out, variant):
    """Rows wider apart than d_in values, with NaN in the gap (own rows and means alike), and NaN rows around the listed
    ones: a kernel that walks such a width as the next multiple of 32 must not let anything beyond a row's d_in values
    into a product, zero weight or not."""
    torch, B = env
    r = np.random.default_rng(d_in * 5 + d_out + variant)
    n_src, n_rows, pad = 1500, 1100, 12
    h = np.full((n_src, d_in + pad), np.nan, np.float32)
    agg = np.full((n_rows, d_in + pad), np.nan, np.float32)
    rows = np.sort(r.permutation(n_src)[:n_rows]).astype(np.int32)
    h[rows, :d_in] = r.standard_normal((n_rows, d_in)).astype(np.float32)
    agg[:, :d_in] = (r.standard_normal((n_rows, d_in)) * 0.3).astype(np.float32)
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    bias = (0.1 * r.standard_normal(d_out)).astype(np.float32)
    t_out = torch.full((n_src, d_out), -3.0, dtype=torch.float32, device="cuda")
    t_cnt = torch.tensor([n_rows], dtype=torch.int64, device="cuda")
    B.fg_set_tuning("linear_tile", variant)
    try:
        B.fg_linear(dev(torch, h), n_src, (d_in + pad) * 4, B.FG_F32, dev(torch, agg), (d_in + pad) * 4, dev(torch, rows), t_cnt,
                    n_rows, d_in, d_out, dev(torch, W), B.FG_F32, dev(torch, bias), 1, t_out, n_src, d_out * 4, B.FG_F32, None)
    finally:
        B.fg_set_tuning("linear_tile", 0)
    got = t_out.cpu().numpy()
    want = O.round_to(O.linear(h[rows, :d_in], agg[:, :d_in], W, bias, True), "f32")
    assert np.all(np.isfinite(got))
    err = T.rel_err_rows(got[rows], want)
    print(f"linear {d_in}x{d_out} with gaps, variant {variant}: rel err {err:.3e}")
    assert err <= REL_TOL_F32


@pytest.mark.parametrize("variant", [0, 8, 32, 64, 301, 302, "bf16", "f16"])
@pytest.mark.parametrize("d_in,d_out,n_rows,max_rows", [(128, 256, 4097, 5000), (256, 256, 700, 700), (100, 64, 333, 400),
                                                        (64, 64, 0, 128), (128, 256, 20000, 20000)])
def test_linear_ids_reads_own_rows_from_the_table(env, d_in, d_out, n_rows, max_rows, variant):
    """fg_linear_ids (own features straight from the table by node id) against the oracle on the gathered rows, and bit for
    bit against fg_linear on a gathered copy; positions whose id is out of range are left alone."""
    torch, B = env
    r = np.random.default_rng(d_in * 13 + d_out + max_rows)
    n_out, table_rows = max_rows + 300, 50_000
    sixteen = variant in ("bf16", "f16")
    if sixteen and d_in % 8:
        pytest.skip("16-bit rows need d_in % 8 == 0")
    src = variant if sixteen else "f32"
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
    code = {"f16": B.FG_F16, "bf16": B.FG_BF16, "f32": B.FG_F32}
    esz = 2 if sixteen else 4
    table = O.round_to(r.standard_normal((table_rows, d_in)), src).astype(np.float32)
    agg = r.standard_normal((max_rows, d_in)) * 0.3
    agg = O.round_bf16(agg) if sixteen else agg.astype(np.float32)
    W = r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)
    W = O.round_bf16(W) if sixteen else W.astype(np.float32)
    bias = (0.1 * r.standard_normal(d_out)).astype(np.float32)
    ids = r.integers(0, table_rows, n_out).astype(np.int32)
    rows = np.sort(r.permutation(n_out)[:max_rows]).astype(np.int32)
    bad = rows[:n_rows][::97]                      # some listed positions carry ids outside the table
    ids[bad[0::2]] = -1
    ids[bad[1::2]] = table_rows
    up = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).cuda().to(tdt[dt])
    t_table, t_agg, t_W = up(table, src), up(agg, "bf16" if sixteen else "f32"), up(W, "bf16" if sixteen else "f32")
    t_cnt = torch.tensor([n_rows], dtype=torch.int64, device="cuda")
    t_out = torch.full((n_out, d_out), -3.0, dtype=torch.float32, device="cuda")
    t_ref = torch.full((n_out, d_out), -3.0, dtype=torch.float32, device="cuda")
    gathered = np.zeros((n_out, d_in), np.float32)
    ok = (ids >= 0) & (ids < table_rows)
    gathered[ok] = table[ids[ok]]
    rows_ok = rows.copy()
    rows_ok[:n_rows][~ok[rows[:n_rows]]] = -1      # what fg_linear needs to be told to skip the same positions
    wcode = B.FG_BF16 if sixteen else B.FG_F32
    B.fg_set_tuning("linear_tile", 0 if sixteen else variant)
    try:
        B.fg_linear_ids(t_table, table_rows, d_in * esz, code[src], dev(torch, ids), t_agg, d_in * esz, dev(torch, rows), t_cnt,
                        max_rows, d_in, d_out, t_W, wcode, dev(torch, bias), 1, t_out, n_out, d_out * 4, B.FG_F32, None)
        B.fg_linear(up(gathered, src), n_out, d_in * esz, code[src], t_agg, d_in * esz, dev(torch, rows_ok), t_cnt,
                    max_rows, d_in, d_out, t_W, wcode, dev(torch, bias), 1, t_ref, n_out, d_out * 4, B.FG_F32, None)
    finally:
        B.fg_set_tuning("linear_tile", 0)
    got, ref = t_out.cpu().numpy(), t_ref.cpu().numpy()
    assert np.array_equal(got, ref)
    sel = rows[:n_rows][ok[rows[:n_rows]]]
    keep = ok[rows[:n_rows]]
    untouched = np.ones(n_out, bool)
    untouched[sel] = False
    assert np.all(got[untouched] == -3.0)
    own = table[ids[sel]]
    want = O.round_to(O.linear(O.round_bf16(own) if sixteen else own, agg[:n_rows][keep], W, bias, True), "f32")
    if len(sel):
        err = T.rel_err_rows(got[sel], want)
        print(f"linear_ids {src} {d_in}x{d_out} rows {n_rows} variant {variant}: rel err {err:.3e}")
        assert err <= (2e-2 if sixteen else REL_TOL_F32)


@pytest.mark.parametrize("d_in,d_out,fan,max_rows,n_rows,listed", [
    (128, 256, 15, 16384, 16384, True), (128, 256, 7, 16421, 16389, True), (100, 252, 15, 17000, 33, True), (4, 4, 3, 16384, 8193, False),
    (64, 88, 15, 20000, 19999, True), (68, 36, 6, 16400, 16400, False), (60, 256, 2, 16384, 0, True), (12, 32, 3, 150000, 149985, True)])
def test_loader_and_dense_update_as_one_launch(env, d_in, d_out, fan, max_rows, n_rows, listed):
    """fg_gather_aggregate_linear_ids where it is one launch, against the means of fg_gather_aggregate_ids multiplied in double (the repository's
    bar): partial blocks, more blocks than a workgroup lists at once, widths that are no multiple of a block's, rows without neighbours and with
    more than a block's row has places for, positions, node ids and ranges that are out of range, a NaN row, outputs beside the listed ones, and a
    fetch of cached rows in the same launch."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import _tensor_from_ptr
    g = torch.Generator(device="cuda").manual_seed(d_in * 7 + n_rows)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=g)
    ints = lambda hi, n: torch.randint(0, hi, (n,), device="cuda", generator=g, dtype=torch.int32)
    table_rows, n_block = 30011, max_rows + 50
    stride = d_in + 4 * (d_in % 8 == 4)                              # rows further apart than they are long, too
    table = rand(table_rows, stride)
    deg = ints(fan + 1, n_block)
    deg[11::1009] = 41
    deg[20] = 2
    end = deg.cumsum(0).to(torch.int32)
    start = (end - deg).to(torch.int32)
    nnz = int(end[-1])
    ids, own = ints(table_rows, nnz), ints(table_rows, n_block)
    ids[ids == 5] = 6                                                # node 5 is the NaN row: a neighbour of one row, its own row of another
    table[5] = float("nan")
    own[own == 5] = 6
    ids[3::1013] = -1
    ids[7::1013] = table_rows
    ids[int(start[20])] = own[30] = 5
    end[40] = start[40] - 1 if int(start[40]) else -1                # no range: a row without neighbours
    rows = torch.arange(n_block, device="cuda", dtype=torch.int32)
    if listed:
        rows = torch.randperm(n_block, device="cuda", generator=g).to(torch.int32)
        own[50] = table_rows                                         # (left alone)
        first = torch.tensor([20, 30, 40, 50], device="cuda", dtype=torch.int32)
        rows = torch.cat([first, rows[~torch.isin(rows, first)]])
        rows[5:7] = torch.tensor([-1, n_block], device="cuda", dtype=torch.int32)
    cnt = torch.tensor([n_rows], dtype=torch.int64, device="cuda")
    W, bias = rand(2 * d_in, d_out) / (2 * d_in) ** 0.5, rand(d_out)
    assert B.one_launch_load(nnz, max_rows, d_in, d_out)
    cache = B.fg_cache_create(1000, [300], [d_out], B.FG_F32, 2, None)
    try:
        cached = _tensor_from_ptr(B.fg_cache_table(cache, 1), (300, d_out), torch.float32, 300 * d_out * 4, "cuda")
        cached.copy_(rand(300, d_out))
        slots, places, n_hit = ints(300, 77), torch.randperm(500, device="cuda")[:77].to(torch.int32), torch.tensor([61], dtype=torch.int64, device="cuda")
        outs = []
        for one in (True, False):
            agg, fetched = torch.full((max_rows, d_in), 7.0, device="cuda"), torch.full((500, d_out), 7.0, device="cuda")
            out = torch.full((n_block, d_out), 7.0, device="cuda")
            specs = B.fetch_layers([dict(layer=1, hit_slot_dev=slots, hit_pos_dev=places, n_hit_dev=n_hit, max_hits=77, h_dev=fetched, h_rows=500,
                                         h_stride=d_out * 4)])
            at = rows if listed else None
            if one:
                B.fg_gather_aggregate_linear_ids(start, end, ids, nnz, n_block, at, cnt, max_rows, own, table, table_rows, stride * 4, d_in, d_out, W, bias, 1,
                                                 agg, d_in * 4, out, n_block, d_out * 4, cache, specs)
            else:
                B.fg_gather_aggregate_ids(start, end, ids, nnz, n_block, at, cnt, max_rows, own, table, table_rows, stride * 4, d_in, B.FG_F32, agg, d_in * 4,
                                          B.FG_F32, None, 0, 0, cache, specs)
            torch.cuda.synchronize()
            outs.append((agg, out, fetched))
    finally:
        B.fg_cache_destroy(cache)
    (_, out1, f1), (agg2, _, f2) = outs
    assert torch.equal(f1, f2) and int((f1 != 7.0).any(1).sum()) == 61
    listed_rows = rows[:n_rows].long()
    good = (listed_rows >= 0) & (listed_rows < n_block)
    r = listed_rows[good]
    ok = (own[r] >= 0) & (own[r] < table_rows)
    r, mean = r[ok], agg2[:n_rows][good][ok]
    x = torch.cat([table[own[r].long(), :d_in], mean], 1).double()
    want = torch.relu(x @ W.double() + bias.double()).cpu().numpy()
    got = out1[r].cpu().numpy()
    bad = ~np.isfinite(x.sum(1).cpu().numpy())
    assert int(bad.sum()) == (2 if n_rows else 0)
    err = T.rel_err_rows(got[~bad], want[~bad]) if (~bad).any() else 0.0
    print(f"loader and dense update {d_in}x{d_out} fan-out {fan} rows {n_rows} of {max_rows}: rel err {err:.3e}")
    assert err <= REL_TOL_F32
    rest = torch.ones(n_block, dtype=torch.bool, device="cuda")
    rest[r] = False
    assert bool((out1[rest] == 7.0).all())


@pytest.mark.parametrize("variant", [0, 301, 302, 32, 64])
@pytest.mark.parametrize("case", ["rows scaled", "mixed within a row", "columns of W scaled", "near the upper limit", "near the lower limit"])
def test_linear_operands_of_mixed_and_extreme_magnitude(env, case, variant):
    """The relative bar is scale-free per row, so it must hold for rows scaled by 2^-60 .. 2^60, for rows whose elements
    differ by 2^40, for weight columns of very different size, and at both ends of the documented input domain
    (magnitudes below 2^127; nonzero magnitudes of at least 2^-100, below which the low bf16 terms of the three-way
    split leave the normal range: tests/test_abi.py models that boundary on the host)."""
    torch, B = env
    r = np.random.default_rng(len(case) * 31 + variant)
    d_in, d_out, n_src, n_rows = 128, 256, 2600, 2100
    h = r.standard_normal((n_src, d_in)).astype(np.float32)
    agg = (r.standard_normal((n_rows, d_in)) * 0.3).astype(np.float32)
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    rows = np.sort(r.permutation(n_src)[:n_rows]).astype(np.int32)
    if case == "rows scaled":
        e = r.integers(-60, 61, n_src)
        h *= np.exp2(e)[:, None].astype(np.float32)
        agg *= np.exp2(e[rows])[:, None].astype(np.float32)
    elif case == "mixed within a row":
        h *= np.exp2(r.integers(-20, 21, h.shape)).astype(np.float32)
        agg *= np.exp2(r.integers(-20, 21, agg.shape)).astype(np.float32)
    elif case == "columns of W scaled":
        W *= np.exp2(r.integers(-30, 31, d_out))[None, :].astype(np.float32)
    elif case == "near the upper limit":
        h *= np.float32(2.0 ** 124)           # |x| up to about 2^126.5
        agg *= np.float32(2.0 ** 124)
        W *= np.float32(2.0 ** -100)          # keeps the outputs finite
    else:
        h *= np.float32(2.0 ** -98)           # most magnitudes in 2^-100 .. 2^-96, a few smaller
        agg *= np.float32(2.0 ** -98)
        W *= np.float32(2.0 ** 60)
    assert np.isfinite(h).all() and np.isfinite(agg).all() and np.isfinite(W).all()
    t_out = torch.zeros((n_src, d_out), dtype=torch.float32, device="cuda")
    t_cnt = torch.tensor([n_rows], dtype=torch.int64, device="cuda")
    B.fg_set_tuning("linear_tile", variant)
    try:
        B.fg_linear(dev(torch, h), n_src, d_in * 4, B.FG_F32, dev(torch, agg), d_in * 4, dev(torch, rows), t_cnt, n_rows, d_in,
                    d_out, dev(torch, W), B.FG_F32, None, 0, t_out, n_src, d_out * 4, B.FG_F32, None)
    finally:
        B.fg_set_tuning("linear_tile", 0)
    got = t_out.cpu().numpy()[rows]
    want = O.round_to(O.linear(h[rows], agg, W, np.zeros(d_out), False), "f32")
    assert np.isfinite(want).all()
    err = T.rel_err_rows(got, want)
    print(f"linear, {case}, variant {variant}: rel err {err:.3e}")
    # Element by element: the relative bar, or, where an output is small next to the terms it is summed from (scaled
    # weight columns leave a row's largest output to a single random sum), 4 fp32 half-ulps of the sum of |terms|
    x64 = np.concatenate([h[rows], agg], axis=1).astype(np.float64)
    terms = np.abs(x64) @ np.abs(W.astype(np.float64))
    ref = np.abs(want.astype(np.float64))
    den = np.maximum(ref, ref.max(axis=1, keepdims=True) / 16.0)
    allowed = np.maximum(REL_TOL_F32 * den, 4 * 2.0 ** -24 * terms)
    excess = np.abs(got.astype(np.float64) - want.astype(np.float64)) - allowed
    assert (excess <= 0).all(), f"{int((excess > 0).sum())} outputs beyond the bound, rel err {err:.3e}"


# ------------------------------------------------------------------------------------------------ fg_cache_update

@pytest.mark.parametrize("cap,t_stale,p,nmax", [(5, 2, 0.5, 12), (64, 4, 0.9, 40), (3, 1, 1.0, 9), (1000, 50, 0.3, 3000),
                                                (4096, 3, 0.7, 5000), (5000, 3, 0.3, 16000), (5000, 2, 0.5, 32000),
                                                (4000, 3, 0.2, 65536), (4500, 2, 0.6, 80000)])
def test_cache_update_sequences_match_oracle(env, cap, t_stale, p, nmax):
    # the list lengths span every variant of the threshold selection (registers: 4096 .. 65536 elements, streamed
    # above that), with a ragged tail, and every fourth update passes misaligned norm and liveness arrays
    torch, B = env
    r = np.random.default_rng(cap + nmax)
    N, d = max(20000, 2 * nmax) if nmax > 100 else 40, 8
    oc = O.HistoricalCache(N, cap, d, t_stale)
    cache = B.fg_cache_create(N, [cap], [d], B.FG_F32, t_stale, None)
    from paper_2301_07482_amd.pipeline import _tensor_from_ptr
    try:
        for i in range(25):
            n = nmax if i == 0 else int(r.integers(nmax // 3 if nmax > 5000 else 0, nmax + 1))
            ids = r.permutation(N)[:n].astype(np.int32)
            live = r.random(n) < 0.8
            gn = np.round(np.exp(r.standard_normal(n)), 1 if nmax < 100 else 3).astype(np.float32)   # ties occur
            rows = r.standard_normal((n, d)).astype(np.float32)
            look = O.lookup_prune(oc, i, ids, live, None, None, None, 0)
            hit_dev, slots_dev, stats_dev = _device_update(torch, B, cache, i, ids, live, gn, p, rows, misalign=i % 4 == 3)
            assert np.array_equal(hit_dev, look["hit"])                       # the device lookup sees the same hits
            assert np.array_equal(slots_dev[:len(look["hit_slot"])], look["hit_slot"])
            st = O.cache_update(oc, i, ids, live, look["hit"], gn, p, rows)
            assert stats_dev == [st["admitted"], st["evicted_by_gradient"], st["overwritten"], st["dropped_overflow"]], \
                f"stats at iteration {i}"
            exp = _export(torch, B, cache, cap, i + 1)
            valid = oc.valid_entries(i + 1) if cap <= 5000 else None
            assert exp["head"] == oc.head
            assert dict(zip(exp["nodes"].tolist(), zip(exp["slots"].tolist(), exp["stamps"].tolist()))) == valid
            tab = _tensor_from_ptr(B.fg_cache_table(cache, 1), (cap, d), torch.float32, cap * d * 4, "cuda").cpu().numpy()
            for v, (s, _) in valid.items():
                assert np.array_equal(tab[s], oc.table[s])
    finally:
        B.fg_cache_destroy(cache)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 4095, 4096, 4097, 6144, 6145, 8187, 8191, 8192, 8193, 12289, 262_144, 262_145])
@pytest.mark.parametrize("p", [0.0, 0.37, 0.75, 1.0])
def test_cache_update_sizes_around_a_workgroups_share(env, n, p):
    """Layers on both sides of what one workgroup takes, and of what workgroups that wait for each other do, cut quads included;
    a ring that some of them wrap, two updates in a row (the second overwrites the first's entries and checks hits out)."""
    _check_update_sizes(env, n, p, lambda r: np.round(np.exp(r.standard_normal(n)), 2))      # ties occur


@pytest.mark.parametrize("n", [4096, 4097, 30_001])
@pytest.mark.parametrize("norms", ["equal", "two values", "one digit apart", "with zeros and infinities"])
def test_cache_update_of_norms_that_share_their_digits(env, n, norms):
    """Thresholds that one, two or all three digits decide, equal keys on both sides of a workgroup's share, and both ends of the range."""
    def draw(r):
        if norms == "equal":
            return np.full(n, 0.7)
        if norms == "two values":
            return np.where(r.random(n) < 0.5, 1.0, 1.0 + 2.0 ** -23)
        if norms == "one digit apart":
            return 1.0 + r.integers(0, 200, n) * 2.0 ** -13
        return np.choose(r.integers(0, 3, n), [np.zeros(n), np.full(n, np.inf), np.exp(r.standard_normal(n))])
    _check_update_sizes(env, n, 0.37, draw)


@pytest.mark.parametrize("n", [4096, 4097, 20_480, 20_481])
def test_cache_update_in_two_parts_on_both_sides_of_its_launches(env, n):
    """fg_cache_update_select and _commit: up to five workgroups of 4096 positions wait for each other, beyond that four launches."""
    _check_update_sizes(env, n, 0.4, lambda r: np.exp(r.standard_normal(n)), two_parts=True)


def _check_update_sizes(env, n, p, norms, two_parts=False):
    torch, B = env
    r = np.random.default_rng(n)
    N, cap, d = max(20000, 3 * n), 4500, 8
    oc = O.HistoricalCache(N, cap, d, 5)
    cache = B.fg_cache_create(N, [cap], [d], B.FG_F32, 5, None)
    try:
        for i in range(2):
            ids = r.permutation(min(N, 2 * n + 8))[:n].astype(np.int32)
            live = r.random(n) < (0.9 if i else 1.1)
            gn = norms(r).astype(np.float32)
            rows = r.standard_normal((n, d)).astype(np.float32)
            look = O.lookup_prune(oc, i, ids, live, None, None, None, 0)
            _, _, stats = _device_update(torch, B, cache, i, ids, live, gn, p, rows, misalign=False, two_parts=two_parts)
            st = O.cache_update(oc, i, ids, live, look["hit"], gn, p, rows)
            assert stats == [st["admitted"], st["evicted_by_gradient"], st["overwritten"], st["dropped_overflow"]]
            exp = _export(torch, B, cache, cap, i + 1)
            assert exp["head"] == oc.head
            assert dict(zip(exp["nodes"].tolist(), zip(exp["slots"].tolist(), exp["stamps"].tolist()))) == oc.valid_entries(i + 1)
    finally:
        B.fg_cache_destroy(cache)


@pytest.mark.parametrize("n", [4097, 30_001, 200_000])
def test_cache_update_whose_workgroups_give_up_changes_no_slot(env, n):
    """Waits of one to three polls: an update either is the one with patient workgroups, or says that its workgroups gave up; then nothing is
    admitted, the ring's header stands, the rows in the cache are those of before, less some check-outs, and the next update is whole."""
    torch, B = env
    r = np.random.default_rng(n)
    N, cap, d = 3 * n, n, 4
    rows = [r.standard_normal((n, d)).astype(np.float32) for _ in range(3)]
    ids = [r.permutation(min(N, 2 * n))[:n].astype(np.int32) for _ in range(3)]
    gn = [np.exp(r.standard_normal(n)).astype(np.float32) for _ in range(3)]
    live = np.ones(n, bool)
    gave_up = 0

    def entries(cache, it):
        e = _export(torch, B, cache, cap, it)
        tab = _table(torch, B, cache, cap, d)
        return e["head"], {int(v): (int(s), int(q), tab[s].tobytes()) for v, s, q in zip(e["nodes"], e["slots"], e["stamps"])}

    def updates(polls):
        cache = B.fg_cache_create(N, [cap], [d], B.FG_F32, 5, None)
        try:
            out = []
            for i in range(3):
                B.fg_set_tuning("wait_polls", polls if i == 1 else 0)
                stats = _device_update(torch, B, cache, i, ids[i], live, gn[i], 0.4, rows[i])[2]
                out.append((stats, *entries(cache, i + 1)))
            return out
        finally:
            B.fg_set_tuning("wait_polls", 0)
            B.fg_cache_destroy(cache)

    whole = updates(0)
    assert all(s[0] > 0 for s, _, _ in whole)
    for trial in range(9):
        got = updates(1 + trial % 3)
        assert got[0] == whole[0]
        if got[1][0][0] >= 0:
            assert got == whole
            continue
        gave_up += 1
        stats, head, there = got[1]
        assert stats[0] == stats[3] == -1 and stats[2] == 0 and head == got[0][1]
        assert there.items() <= got[0][2].items() and len(there) >= len(got[0][2]) - stats[1]
        hit = np.asarray([int(v) in there for v in ids[2]])
        low = gn[2] < np.sort(gn[2])[int(np.floor(np.float32(0.4) * n))]
        assert got[2][0][0] == min(cap, int((low & ~hit).sum())) and got[2][0][1] == int((~low & hit).sum())
    print(f"{gave_up} of 9 gave up")


@pytest.mark.parametrize("n,d,p", [(1, 4, 1.0), (4096, 4, 1.0), (777, 12, 0.6), (1024, 64, 0.6), (3000, 20, 0.5), (4096, 20, 0.5),      # copied by the selection
                                   (1024, 64, 0.8), (4096, 20, 0.51), (1024, 64, 0.9), (4096, 28, 0.6), (4097, 4, 0.3)])                               # by a launch of their own
def test_cache_update_rows_of_small_layers(env, n, d, p):
    """The rows a small layer's update puts into the cache, on both sides of the size up to which the selecting workgroup copies
    them itself; a ring that wraps, rows of 16 to 256 bytes."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import _tensor_from_ptr
    r = np.random.default_rng(n + d)
    N, cap = 9000, max(2, n // 2 + 3)
    oc = O.HistoricalCache(N, cap, d, 5)
    cache = B.fg_cache_create(N, [cap], [d], B.FG_F32, 5, None)
    try:
        for i in range(2):
            ids = r.permutation(N)[:n].astype(np.int32)
            live, gn = np.ones(n, bool), np.exp(r.standard_normal(n)).astype(np.float32)
            rows = r.standard_normal((n, d)).astype(np.float32)
            look = O.lookup_prune(oc, i, ids, live, None, None, None, 0)
            _device_update(torch, B, cache, i, ids, live, gn, p, rows)
            O.cache_update(oc, i, ids, live, look["hit"], gn, p, rows)
            tab = _tensor_from_ptr(B.fg_cache_table(cache, 1), (cap, d), torch.float32, cap * d * 4, "cuda").cpu().numpy()
            at = {int(v): k for k, v in enumerate(ids)}
            new = [(slot, at[node]) for node, (slot, stamp) in oc.valid_entries(i + 1).items() if stamp == i]
            assert len(new) == min(cap, int(np.floor(np.float32(p) * n)) if p < 1 else n) or i > 0
            assert all(np.array_equal(tab[slot], rows[k]) for slot, k in new)
    finally:
        B.fg_cache_destroy(cache)


def _export(torch, B, cache, cap, it, layer=1):
    t = [torch.zeros(cap, dtype=torch.int32, device="cuda") for _ in range(3)]
    cnt = torch.zeros(2, dtype=torch.int64, device="cuda")
    wsb = B.fg_workspace_bytes(B.FG_WS_EXPORT, cap)
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    B.fg_cache_export(cache, layer, it, t[0], t[1], t[2], cnt.data_ptr(), cnt.data_ptr() + 8, ws, wsb, None)
    c = int(cnt[0].item())
    return dict(nodes=t[0][:c].cpu().numpy(), slots=t[1][:c].cpu().numpy(), stamps=t[2][:c].cpu().numpy(), head=int(cnt[1].item()))


def _table(torch, B, cache, cap, d):
    from paper_2301_07482_amd.pipeline import _tensor_from_ptr
    return _tensor_from_ptr(B.fg_cache_table(cache, 1), (cap, d), torch.float32, cap * d * 4, "cuda").cpu().numpy()


def test_iteration_counter_must_not_go_backwards(env):
    torch, B = env
    cache = B.fg_cache_create(100, [10], [4], B.FG_F32, 3, None)
    try:
        z = lambda dt, n=4: torch.zeros(n, dtype=dt, device="cuda")
        ws = torch.zeros(B.fg_workspace_bytes(B.FG_WS_CACHE_UPDATE, 4), dtype=torch.uint8, device="cuda")
        args = lambda it: (cache, 1, it, dev(torch, np.arange(4, dtype=np.int32)), 4, None, z(torch.uint8), z(torch.float32),
                           0.5, torch.zeros((4, 4), device="cuda"), 16, None, ws, ws.numel(), None)
        B.fg_cache_update(*args(5))
        with pytest.raises(B.FgError) as e:
            B.fg_cache_update(*args(4))
        assert e.value.code == B.FG_ERR_STATE
    finally:
        B.fg_cache_destroy(cache)


def test_update_all_and_fetch_all_with_unequal_and_empty_layers(env):
    """fg_cache_update_all / fg_cache_fetch_all over three layers of very different sizes, one of them empty in some
    iterations, against the oracle's per-layer updates: cache state, statistics and fetched rows."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import _tensor_from_ptr
    r = np.random.default_rng(77)
    N, dims, caps, t_stale, p = 30000, [8, 16, 4], [300, 5000, 64], 3, 0.6
    oc = [O.HistoricalCache(N, caps[k], dims[k], t_stale) for k in range(3)]
    cache = B.fg_cache_create(N, caps, dims, B.FG_F32, t_stale, None)
    try:
        for i in range(12):
            ns = [int(r.integers(0, 400)) if i % 3 else 0, int(r.integers(3000, 9000)), int(r.integers(1, 90))]
            ids = [r.permutation(N)[:n].astype(np.int32) for n in ns]
            live = [r.random(n) < 0.85 for n in ns]
            gn = [np.round(np.exp(r.standard_normal(n)), 2).astype(np.float32) for n in ns]
            rows = [r.standard_normal((n, dims[k])).astype(np.float32) for k, n in enumerate(ns)]
            look = [O.lookup_prune(oc[k], i, ids[k], live[k], None, None, None, 0) for k in range(3)]
            # device lookups (per layer), then one fetch call and one update call for all three layers
            t_ids = [dev(torch, a) for a in ids]
            t_live = [dev(torch, a.astype(np.uint8)) for a in live]
            t_hit = [torch.zeros(max(n, 1), dtype=torch.uint8, device="cuda") for n in ns]
            t_pos = [torch.zeros(max(n, 1), dtype=torch.int32, device="cuda") for n in ns]
            t_slot = [torch.zeros(max(n, 1), dtype=torch.int32, device="cuda") for n in ns]
            t_norm = [torch.zeros(max(n, 1), dtype=torch.int32, device="cuda") for n in ns]
            t_cnt = torch.zeros((3, 3), dtype=torch.int64, device="cuda")
            for k in range(3):
                wsb = B.fg_workspace_bytes(B.FG_WS_LOOKUP_PRUNE, ns[k])
                ws = torch.zeros(max(wsb, 16), dtype=torch.uint8, device="cuda")
                B.fg_lookup_prune(cache, k + 1, i, t_ids[k], ns[k], t_live[k], None, None, None, 0, 0, None, t_hit[k], t_pos[k],
                                  t_slot[k], t_norm[k], None, t_cnt[k], ws, wsb, None)
            t_H = [torch.full((max(n, 1), dims[k]), -5.0, device="cuda") for k, n in enumerate(ns)]
            B.fg_cache_fetch_all(cache, B.fetch_layers([dict(layer=k + 1, hit_slot_dev=t_slot[k], hit_pos_dev=t_pos[k],
                                                             n_hit_dev=t_cnt[k].data_ptr() + 8, max_hits=ns[k], h_dev=t_H[k],
                                                             h_rows=ns[k], h_stride=dims[k] * 4) for k in range(3)]), None)
            for k in range(3):
                got = t_H[k].cpu().numpy()[:ns[k]]
                assert np.array_equal(t_hit[k].cpu().numpy()[:ns[k]].astype(bool), look[k]["hit"])
                want = np.full((ns[k], dims[k]), -5.0, np.float32)
                if len(look[k]["hit_pos"]):
                    want[look[k]["hit_pos"]] = oc[k].table[look[k]["hit_slot"]]
                assert np.array_equal(got, want), f"fetched rows of layer {k + 1} at iteration {i}"
            t_rows = [dev(torch, a) if a.size else torch.zeros((1, dims[k]), device="cuda") for k, a in enumerate(rows)]
            t_gn = [dev(torch, a) if a.size else torch.zeros(1, device="cuda") for a in gn]
            t_stats = torch.zeros((3, 4), dtype=torch.int64, device="cuda")
            wsb = sum(B.fg_workspace_bytes(B.FG_WS_CACHE_UPDATE, n) for n in ns)
            ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
            specs = B.update_layers([dict(layer=k + 1, n=ns[k], ids_dev=t_ids[k], live_dev=t_live[k], hit_dev=t_hit[k],
                                          gnorm_dev=t_gn[k], h_dev=t_rows[k], h_stride=dims[k] * 4, stats_dev=t_stats[k].data_ptr())
                                     for k in range(3)])
            if i % 2:       # the same update in two calls; in between the cache refuses further updates
                B.fg_cache_update_select(cache, i, p, specs, ws, wsb, None)
                for call in (lambda: B.fg_cache_update_all(cache, i, p, specs, ws, wsb, None),
                             lambda: B.fg_cache_update_select(cache, i, p, specs, ws, wsb, None),
                             lambda: B.fg_cache_update_commit(cache, i + 1, specs, ws, wsb, None)):
                    with pytest.raises(B.FgError) as e:
                        call()
                    assert e.value.code == B.FG_ERR_STATE
                B.fg_cache_update_commit(cache, i, specs, ws, wsb, None)
                with pytest.raises(B.FgError) as e:
                    B.fg_cache_update_commit(cache, i, specs, ws, wsb, None)       # nothing is waiting any more
                assert e.value.code == B.FG_ERR_STATE
            else:
                B.fg_cache_update_all(cache, i, p, specs, ws, wsb, None)
            stats = t_stats.cpu().numpy().tolist()
            for k in range(3):
                st = O.cache_update(oc[k], i, ids[k], live[k], look[k]["hit"], gn[k], p, rows[k])
                assert stats[k] == [st["admitted"], st["evicted_by_gradient"], st["overwritten"], st["dropped_overflow"]], \
                    f"stats of layer {k + 1} at iteration {i}"
                exp = _export(torch, B, cache, caps[k], i + 1, layer=k + 1)
                valid = oc[k].valid_entries(i + 1)
                assert exp["head"] == oc[k].head
                assert dict(zip(exp["nodes"].tolist(), zip(exp["slots"].tolist(), exp["stamps"].tolist()))) == valid
                tab = _tensor_from_ptr(B.fg_cache_table(cache, k + 1), (caps[k], dims[k]), torch.float32, caps[k] * dims[k] * 4,
                                       "cuda").cpu().numpy()
                for v, (s, _) in valid.items():
                    assert np.array_equal(tab[s], oc[k].table[s])
    finally:
        B.fg_cache_destroy(cache)


# ------------------------------------------------------------------------------------------------ device-side sampler

def _random_multigraph(num_nodes, max_deg, seed, hubs=0):
    """In-neighbour CSR with self loops, repeated neighbours, isolated nodes and a few very wide rows."""
    r = np.random.default_rng(seed)
    deg = r.integers(0, max_deg + 1, size=num_nodes)
    deg[r.integers(0, num_nodes, size=hubs)] = r.integers(500, 3000, size=hubs)
    indptr = np.zeros(num_nodes + 1, dtype=np.int64)
    indptr[1:] = np.cumsum(deg)
    near = (np.repeat(np.arange(num_nodes), deg) + r.integers(-4, 5, size=int(indptr[-1]))) % num_nodes
    far = r.integers(0, num_nodes, size=int(indptr[-1]))
    indices = np.where(r.random(int(indptr[-1])) < 0.5, near, far).astype(np.int32)
    return indptr, indices


def _device_sample(torch, B, indptr_t, indices_t, N, seeds, fanouts, key, slack=0):
    """All blocks of a mini-batch through fg_sample_block, each layer's device-side count feeding the next call."""
    L = len(fanouts)
    out = dict(ids=[None] * (L + 1), start=[None] * (L + 1), end=[None] * (L + 1), col=[None] * (L + 1), col_ids=[None] * (L + 1))
    bound = len(seeds) + slack
    cur = torch.zeros(max(bound, 1), dtype=torch.int32, device="cuda")
    cur[:len(seeds)] = dev(torch, np.asarray(seeds, dtype=np.int32))
    n_dev = torch.tensor([len(seeds)], dtype=torch.int64, device="cuda")
    out["ids"][L] = [int(v) for v in seeds]
    for l in range(L, 0, -1):
        f = int(fanouts[l - 1])
        below_bound = bound * (1 + f)
        start = torch.full((max(bound, 1),), -3, dtype=torch.int32, device="cuda")
        end = torch.full((max(bound, 1),), -3, dtype=torch.int32, device="cuda")
        col = torch.full((max(bound * f, 1),), -3, dtype=torch.int32, device="cuda")
        col_ids = torch.full((max(bound * f, 1),), -3, dtype=torch.int32, device="cuda") if l % 2 else None
        below = torch.full((max(below_bound, 1),), -3, dtype=torch.int32, device="cuda")
        counts = torch.full((2,), -3, dtype=torch.int64, device="cuda")
        wsb = B.fg_sample_block_workspace_bytes(bound, f)
        ws = torch.zeros(max(wsb, 16), dtype=torch.uint8, device="cuda")
        B.fg_sample_block(indptr_t, indices_t, N, int(indices_t.numel()), cur, n_dev, bound, f, key, l, start, end, col, col_ids,
                          below, below_bound, counts, ws, wsb)
        n = int(n_dev.item())
        nb, nnz = (int(x) for x in counts.cpu().tolist())
        out["start"][l], out["end"][l] = start.cpu().numpy()[:n].tolist(), end.cpu().numpy()[:n].tolist()
        assert start.cpu().numpy()[n:bound].tolist() == [nnz] * (bound - n) == end.cpu().numpy()[n:bound].tolist()
        out["col"][l] = col.cpu().numpy()[:nnz].tolist()
        out["col_ids"][l] = col_ids.cpu().numpy()[:nnz].tolist() if col_ids is not None else None
        out["ids"][l - 1] = below.cpu().numpy()[:nb].tolist()
        cur, n_dev, bound = below, counts[:1].clone(), below_bound
    return out


@pytest.mark.parametrize("N,max_deg,hubs,n_seeds,fanouts,slack,seed", [
    (50, 6, 0, 9, (3, 2), 0, 0), (400, 40, 5, 40, (10, 5), 3, 1), (30000, 60, 40, 700, (15, 10, 5), 100, 2),
    (2000, 100, 10, 300, (32, 1), 0, 3), (500, 3, 0, 0, (4, 4), 5, 4), (5000, 45, 20, 1100, (25, 15), 0, 5)])
def test_sample_block_matches_oracle(env, N, max_deg, hubs, n_seeds, fanouts, slack, seed):
    """fg_sample_block, layer after layer on device-side counts, against the oracle's sampler: node lists, row bounds,
    columns as positions and as ids, counts; bit for bit. Graphs with self loops, repeated neighbours, isolated nodes and
    rows far wider than the fan-out; fan-outs 1 and 32; no seeds; bounds larger than the counts."""
    torch, B = env
    from oracle import sampler_oracle as S
    indptr, indices = _random_multigraph(N, max_deg, seed, hubs)
    indptr_t, indices_t = dev(torch, indptr), dev(torch, indices) if len(indices) else torch.zeros(1, dtype=torch.int32, device="cuda")
    r = np.random.default_rng(seed)
    for rep in range(3):
        seeds = r.permutation(N)[:n_seeds]
        key = int(r.integers(0, 2 ** 62))
        want = S.sample_minibatch(indptr, indices, seeds, fanouts, key)
        got = _device_sample(torch, B, indptr_t, indices_t, N, seeds, fanouts, key, slack)
        L = len(fanouts)
        for l in range(L, 0, -1):
            assert got["ids"][l - 1] == want["ids"][l - 1], f"nodes of layer {l - 1}"
            assert got["start"][l] == want["start"][l] and got["end"][l] == want["end"][l], f"rows of block {l}"
            assert got["col"][l] == want["col"][l], f"columns of block {l}"
            if got["col_ids"][l] is not None:
                assert got["col_ids"][l] == want["col_ids"][l]


@pytest.mark.parametrize("N,max_deg,n_seeds,fanout,bound,seed", [
    (9000, 30, 1024, 11, 1024, 0), (9000, 30, 1023, 11, 1024, 1),      # nearly every draw new
    (9000, 30, 1025, 11, 1025, 2), (9000, 30, 1000, 12, 1000, 3),       # one row, one draw more
    (9000, 30, 512, 11, 512, 12), (9000, 30, 704, 8, 704, 13), (9000, 30, 1024, 5, 1024, 14), (9000, 30, 700, 8, 704, 15),
    (9000, 30, 513, 11, 513, 16), (9000, 30, 1024, 6, 1024, 17), (9000, 30, 704, 8, 705, 18),
    (9000, 30, 1024, 7, 1024, 19), (9000, 30, 890, 8, 896, 20), (9000, 30, 651, 11, 651, 21),      # the most draws of one workgroup
    (9000, 30, 1024, 8, 1024, 23), (9000, 30, 896, 8, 897, 22), (9000, 30, 652, 11, 652, 24),      # and more
    (40, 60, 40, 11, 1024, 4), (3000, 3, 1, 1, 1, 5), (3000, 40, 0, 5, 7, 6),      # many repeats, one row, none
    (5000, 50, 1500, 8, 1501, 7), (5000, 50, 1500, 9, 1600, 8), (5000, 50, 1500, 16, 1500, 9), (5000, 50, 1500, 17, 1500, 10),
    (4000, 40, 2600, 15, 600_000, 11), (4000, 40, 300, 32, 1_048_577, 31),     # (the second: beyond what a workgroup adds up for itself)
    (9000, 30, 512, 8, 512, 25), (9000, 30, 512, 8, 513, 26), (9000, 30, 372, 11, 372, 27),      # one workgroup up to 4096 draws
    (6000, 40, 5000, 15, 34_816, 28), (6000, 40, 5000, 15, 34_817, 29), (6000, 40, 5000, 1, 524_289, 30)])   # one slot per thread or four
def test_sample_block_routes_match_oracle(env, N, max_deg, n_seeds, fanout, bound, seed):
    """One block at the sizes where fg_sample_block changes its launches (one workgroup or several, one slot per thread or four,
    the workgroups' counts added up by each or once), bit for bit."""
    torch, B = env
    from oracle import sampler_oracle as S
    indptr, indices = _random_multigraph(N, max_deg, seed, hubs=3)
    seeds = np.random.default_rng(seed).permutation(N)[:n_seeds]
    want = S.sample_minibatch(indptr, indices, seeds, (fanout,), 77 + seed)
    got = _device_sample(torch, B, dev(torch, indptr), dev(torch, indices), N, seeds, (fanout,), 77 + seed, bound - n_seeds)
    for key, l in (("ids", 0), ("start", 1), ("end", 1), ("col", 1), ("col_ids", 1)):
        assert got[key][l] == want[key][l], key


@pytest.mark.parametrize("N,max_deg,hubs,batch,n_seeds,fanouts,seed", [
    (9000, 30, 3, 200, 200, (3, 4, 5), 0),          # the seeds' block by one workgroup, its transpose rides behind it
    (9000, 30, 3, 1024, 1000, (10, 5), 1),          # ... by three launches, fewer seeds than the bound
    (300, 30, 40, 64, 64, (10, 10), 2),             # both blocks by one workgroup, few nodes
    (6000, 40, 20, 1100, 1100, (15, 32), 3),        # four slots per thread
    (20000, 8, 3, 16385, 16384, (32,), 8),          # four slots in the bound, one in the call
    (6000, 40, 3, 4100, 700, (2, 32), 4),           # more than 131 072 sources: four stages for three launches
    (3000, 20, 3, 5, 5, (1,) * 10, 5), (3000, 20, 3, 40, 40, (7,), 6), (3000, 20, 3, 8, 0, (3, 2, 2), 7)])
def test_sample_minibatch_matches_oracle(env, N, max_deg, hubs, batch, n_seeds, fanouts, seed):
    """fg_sample_minibatch with the transposes riding in the next block's launches, two mini-batches behind each other in the same
    workspace and memory, against the oracle's sampler and transpose, bit for bit."""
    torch, B = env
    from oracle import sampler_oracle as S
    from paper_2301_07482_amd.pipeline import DeviceSampler
    indptr, indices = _random_multigraph(N, max_deg, seed, hubs)
    sampler = DeviceSampler(dev(torch, indptr), dev(torch, indices), N, fanouts, batch, transposes=True)
    r, L, out = np.random.default_rng(seed), len(fanouts), sampler.buffers()
    for rep in range(2):
        seeds, key = r.permutation(N)[:n_seeds], int(r.integers(0, 2 ** 62))
        want = S.sample_minibatch(indptr, indices, seeds, fanouts, key)
        bt = sampler.sample(dev(torch, seeds.astype(np.int32)), key, out=out)
        for l in range(L, 0, -1):
            n, nb, nnz = bt.n[l], bt.n[l - 1], bt.nnz[l]
            assert (n, nb, nnz) == (len(want["ids"][l]), len(want["ids"][l - 1]), len(want["col"][l]))
            assert bt.ids[l - 1].cpu().numpy()[:nb].tolist() == want["ids"][l - 1], f"nodes of layer {l - 1}"
            for name in ("start", "end"):
                assert getattr(bt, name)[l].cpu().numpy()[:n].tolist() == want[name][l], f"rows of block {l}"
            assert bt.col[l].cpu().numpy()[:nnz].tolist() == want["col"][l], f"columns of block {l}"
            if l == 1:
                assert bt.col_ids1.cpu().numpy()[:nnz].tolist() == want["col_ids"][1]
            if l >= 2:
                t = S.transpose_block(want["start"][l], want["end"][l], want["col"][l], nb)
                assert [x[l].cpu().numpy()[:m].tolist() for x, m in ((bt.t_start, nb), (bt.t_end, nb), (bt.t_row, nnz))] == [list(x) for x in t], \
                    f"transpose of block {l}"


@pytest.mark.parametrize("first,empty", [((100, 600), [(50, True)]), ((0, 200_000), [(50, True)]), ((100, 600), [(200_000, True), (50, True), (7, False)])])
def test_sample_minibatch_with_an_empty_block_behind_another(env, first, empty):
    """A block without rows has fewer transpose stages than what is left of the block before it, and no launches of its own: the lists of
    both are complete, those of the empty one empty, and the call ends."""
    torch, B = env
    from oracle import sampler_oracle as S
    N, fanout, key = 3000, 5, 99
    indptr, indices = _random_multigraph(N, 20, 1, hubs=2)
    rows, below = first
    seeds = np.random.default_rng(0).permutation(N)[:rows]
    full = lambda n, v=-3, dt=torch.int32: torch.full((max(n, 1),), v, dtype=dt, device="cuda")
    out, specs = [], []
    for i, (r, nb, tr) in enumerate([(rows, below, True)] + [(0, nb, tr) for nb, tr in empty]):
        o = dict(row_start_dev=full(r), row_end_dev=full(r), col_dev=full(r * fanout), ids_below_dev=full(nb), counts_dev=full(2, dt=torch.int64))
        if tr:
            o.update(t_start_dev=full(nb), t_end_dev=full(nb), t_row_dev=full(r * fanout))
        out.append(o)
        specs.append(dict(o, layer=9 - i, fanout=fanout, max_rows=r, max_below=nb))
    layers = B.sample_layers(specs)
    wsb = B.fg_sample_minibatch_workspace_bytes(layers)
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    B.fg_sample_minibatch(dev(torch, indptr), dev(torch, indices), N, len(indices), dev(torch, seeds.astype(np.int32)) if rows else full(1), None, layers, key,
                          ws, wsb)
    torch.cuda.synchronize()
    for o, (nb, tr) in zip(out[1:], empty):
        assert o["counts_dev"].tolist() == [0, 0]
        if tr:
            assert not o["t_start_dev"].any() and not o["t_end_dev"].any()
    if rows == 0:
        assert out[0]["counts_dev"].tolist() == [0, 0] and not out[0]["t_start_dev"].any() and not out[0]["t_end_dev"].any()
        return
    nb, nnz = out[0]["counts_dev"].tolist()
    start, end, col = (out[0][k].cpu().numpy()[:m].tolist() for k, m in (("row_start_dev", rows), ("row_end_dev", rows), ("col_dev", nnz)))
    t = S.transpose_block(start, end, col, nb)
    assert [out[0][k].cpu().numpy()[:m].tolist() for k, m in (("t_start_dev", nb), ("t_end_dev", nb), ("t_row_dev", nnz))] == [list(x) for x in t]


def test_sampler_writes_into_memory_larger_than_it_needs(env):
    """`out` of another sampler, which was made for larger mini-batches: the arrays lie at its front, what is behind stays as it is."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import DeviceSampler
    N = 3000
    indptr, indices = _random_multigraph(N, 20, 3, hubs=2)
    args = (dev(torch, indptr), dev(torch, indices), N)
    small, large = DeviceSampler(*args, (4, 3), 20, transposes=True), DeviceSampler(*args, (4, 3), 50, transposes=True)
    seeds = dev(torch, np.arange(20, dtype=np.int32))
    buf, counts = large.buffers()
    buf.fill_(-5)
    got, want = small.sample(seeds, 7, out=(buf, counts)), small.sample(seeds, 7)
    for name in ("start", "end", "col", "ids", "t_start", "t_end", "t_row"):
        for l in range(3):
            a, b = getattr(got, name)[l], getattr(want, name)[l]
            n = want.nnz[l] if name in ("col", "t_row") else want.n[l - 1] if name.startswith("t_") else want.n[l]
            assert (a is None) == (b is None) and (a is None or torch.equal(a[:n], b[:n])), (name, l)
    assert (buf[small.out_elems:] == -5).all()


@pytest.mark.parametrize("n,n_src,deg,src_bound,nnz_bound", [
    (1500, 12288, 8, 12288, 12288), (1500, 12288, 8, 12288, 12289), (1500, 12288, 8, 12289, 12288), (2500, 5, 4, 9, 12000),
    (1024, 7168, 7, 7168, 7168), (1024, 7168, 7, 7168, 7169), (1024, 7168, 7, 7169, 7168), (1536, 6000, 4, 7168, 7168),
    (1537, 6000, 4, 7168, 7168), (1400, 5, 4, 9, 7000),
    (1, 1, 1, 1, 1), (900, 7000, 21, 131_073, 20_000), (900, 7000, 21, 131_072, 20_000)])
def test_transpose_block_routes(env, n, n_src, deg, src_bound, nnz_bound):
    """The transpose at the sizes where fg_transpose_block changes its launches: one workgroup or several, counters added up
    directly or through per-workgroup sums. Every row names `deg` sources; few sources make lists of thousands."""
    torch, B = env
    from oracle import sampler_oracle as S
    r = np.random.default_rng(n)
    start, end = (np.arange(n) * deg).astype(np.int32), (np.arange(n) * deg + deg).astype(np.int32)
    col = r.integers(0, n_src, size=n * deg).astype(np.int32)
    want = S.transpose_block(start, end, col, n_src)
    t_start, t_end = (torch.full((src_bound,), -3, dtype=torch.int32, device="cuda") for _ in range(2))
    t_row = torch.full((nnz_bound,), -3, dtype=torch.int32, device="cuda")
    cnt = torch.tensor([n, n_src], dtype=torch.int64, device="cuda")
    wsb = B.fg_transpose_block_workspace_bytes(src_bound)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    col_t = torch.zeros(nnz_bound, dtype=torch.int32, device="cuda")
    col_t[:len(col)] = dev(torch, col)
    B.fg_transpose_block(dev(torch, start), dev(torch, end), col_t, cnt.data_ptr(), n, cnt.data_ptr() + 8, src_bound, nnz_bound,
                         t_start, t_end, t_row, ws, wsb)
    assert t_start.cpu().numpy()[:n_src].tolist() == want[0] and t_end.cpu().numpy()[:n_src].tolist() == want[1]
    assert t_row.cpu().numpy()[:n * deg].tolist() == want[2] and set(t_row.cpu().numpy()[n * deg:].tolist()) <= {-3}
    assert set(t_start.cpu().numpy()[n_src:].tolist() + t_end.cpu().numpy()[n_src:].tolist()) <= {n * deg}


@pytest.mark.parametrize("n,n_src,max_deg,slack,seed", [(0, 4, 3, 2, 0), (1, 1, 0, 0, 1), (700, 3000, 12, 50, 2), (6000, 40000, 15, 0, 3),
                                                        (3000, 40, 10, 7, 4)])
def test_transpose_block_matches_oracle(env, n, n_src, max_deg, slack, seed):
    """fg_transpose_block against the oracle's definition, bit for bit: rows pruned in between, bounds larger than the
    device-side counts, sources sampled by hundreds of rows (40 sources for 3000 rows), an empty block."""
    torch, B = env
    from oracle import sampler_oracle as S
    r = np.random.default_rng(seed)
    deg = r.integers(0, max_deg + 1, size=n)
    gap = r.integers(0, 3, size=n)
    start = (np.cumsum(deg + gap) - deg - gap).astype(np.int32)
    end = (start + deg).astype(np.int32)
    nnz = int((deg + gap).sum())
    col = r.integers(0, max(n_src, 1), size=nnz).astype(np.int32)
    want = S.transpose_block(start, end, col, n_src)
    rows_b, src_b = n + slack, n_src + slack
    pad = lambda a, m: dev(torch, np.concatenate([a, np.full(m - len(a), 7, dtype=np.int32)])) if m else torch.zeros(1, dtype=torch.int32, device="cuda")
    t_start = torch.full((max(src_b, 1),), -3, dtype=torch.int32, device="cuda")
    t_end = torch.full((max(src_b, 1),), -3, dtype=torch.int32, device="cuda")
    t_row = torch.full((max(nnz, 1),), -3, dtype=torch.int32, device="cuda")
    cnt = torch.tensor([n, n_src], dtype=torch.int64, device="cuda")
    wsb = B.fg_transpose_block_workspace_bytes(src_b)
    ws = torch.zeros(max(wsb, 16), dtype=torch.uint8, device="cuda")
    B.fg_transpose_block(pad(start, rows_b), pad(end, rows_b), dev(torch, col) if nnz else None, cnt.data_ptr(), rows_b,
                         cnt.data_ptr() + 8, src_b, nnz, t_start, t_end, t_row, ws, wsb)
    total = len(want[2])
    assert t_start.cpu().numpy()[:n_src].tolist() == want[0] and t_end.cpu().numpy()[:n_src].tolist() == want[1]
    assert t_row.cpu().numpy()[:total].tolist() == want[2]
    assert t_start.cpu().numpy()[n_src:src_b].tolist() == [total] * slack == t_end.cpu().numpy()[n_src:src_b].tolist()


@pytest.mark.parametrize("twice", [False, True])
@pytest.mark.parametrize("n,pad", [(700, 0), (700, 20_000), (8192, 20_000), (8193, 20_000), (131_072, 0), (131_073, 0)])
def test_transpose_sorts_lists_by_length(env, n, pad, twice):
    """Sources sampled by 1 to 700 rows (the lengths and sizes of a block at which another sort takes over, by one workgroup and by
    several); twice: some rows name such a source twice."""
    torch, B = env
    from oracle import sampler_oracle as S
    r = np.random.default_rng(n + pad)
    lens = [1, 2, 7, 8, 9, 10, 63, 64, 65, 66, 128, 257, 700] * 3 + [0] * 5 + [3] * 1200
    rows = [r.permutation(n)[:m] for m in lens]
    if twice:
        rows = [np.concatenate([x, x[:2]]) if j % 2 and len(x) > 8 else x for j, x in enumerate(rows)]
    src = np.repeat(np.arange(len(lens)), [len(x) for x in rows])
    rows = np.concatenate(rows)
    order = r.permutation(len(rows))
    order = order[np.argsort(rows[order], kind="stable")]      # a row's sources in any order
    col = src[order].astype(np.int32)
    end = np.cumsum(np.bincount(rows, minlength=n)).astype(np.int32)
    start = np.concatenate([[0], end[:-1]]).astype(np.int32)
    want = S.transpose_block(start, end, col, len(lens))
    nnz = len(col) + pad
    t_start, t_end = (torch.zeros(len(lens), dtype=torch.int32, device="cuda") for _ in range(2))
    t_row = torch.zeros(nnz, dtype=torch.int32, device="cuda")
    wsb = B.fg_transpose_block_workspace_bytes(len(lens))
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    col_t = dev(torch, np.concatenate([col, np.zeros(pad, dtype=np.int32)]))
    B.fg_transpose_block(dev(torch, start), dev(torch, end), col_t, None, n, None, len(lens), nnz, t_start, t_end, t_row, ws, wsb)
    assert t_start.tolist() == want[0] and t_end.tolist() == want[1] and t_row.tolist()[:len(col)] == want[2]


# ------------------------------------------------------------------------------------------------ access-aware admission

@pytest.mark.parametrize("n,n_src,max_deg,seed", [(0, 5, 3, 0), (1, 1, 0, 1), (700, 3000, 12, 2), (5000, 40000, 30, 3), (300, 300, 2500, 4)])
def test_access_estimate_matches_oracle(env, n, n_src, max_deg, seed):
    """fg_access_estimate against the oracle, bit for bit: the input layer below (NULL) and estimates below, hits,
    pruned rows, saturation (rows of up to 2500 neighbours and estimates beyond 2047 below)."""
    torch, B = env
    r = np.random.default_rng(seed)
    deg = r.integers(0, max_deg + 1, size=n)
    gap = r.integers(0, 3, size=n)                                   # unused columns between rows, as pruning leaves them
    start = (np.cumsum(deg + gap) - deg - gap).astype(np.int32)
    end = (start + deg).astype(np.int32)
    pruned = r.random(n) < 0.2
    end[pruned] = start[pruned]
    nnz = int((deg + gap).sum())
    col = r.integers(0, max(n_src, 1), size=nnz).astype(np.int32)
    hit = r.random(n) < 0.25
    for below in (None, r.integers(1, 40, size=n_src).astype(np.int32), r.integers(1, 5000, size=n_src).astype(np.int32)):
        want = O.access_estimate(start, end, col, hit, below)
        out = torch.full((max(n, 1),), -7, dtype=torch.int32, device="cuda")
        B.fg_access_estimate(dev(torch, start) if n else None, dev(torch, end) if n else None, dev(torch, col) if nnz else None, nnz, n,
                             dev(torch, hit.astype(np.uint8)) if n else None, None if below is None else dev(torch, below), n_src, out)
        assert np.array_equal(out.cpu().numpy()[:n], want)
        if n:      # no hit flags: every row is computed
            want = O.access_estimate(start, end, col, np.zeros(n, dtype=bool), below)
            B.fg_access_estimate(dev(torch, start), dev(torch, end), dev(torch, col) if nnz else None, nnz, n, None,
                                 None if below is None else dev(torch, below), n_src, out)
            assert np.array_equal(out.cpu().numpy()[:n], want)


def test_access_aware_admission_matches_oracle(env):
    """fg_cache_update_all with estimates and budgets against the oracle's rule, three layers in one call: a budget that
    changes every update with few distinct estimates (many ties at the threshold), estimates beyond the saturation point
    with only the ring's capacity as the limit, and a budget without estimates (position order). Cache state, statistics
    and stored rows, bit for bit."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import _tensor_from_ptr
    r = np.random.default_rng(91)
    N, dims, caps, t_stale, p = 30000, [8, 16, 4], [4000, 900, 300], 3, 0.8
    oc = [O.HistoricalCache(N, caps[k], dims[k], t_stale) for k in range(3)]
    cache = B.fg_cache_create(N, caps, dims, B.FG_F32, t_stale, None)
    turned_away = [0, 0, 0]
    try:
        for i in range(14):
            ns = [int(r.integers(2000, 9000)), int(r.integers(1500, 3000)), int(r.integers(0, 700)) if i % 4 else 0]
            ids = [r.permutation(N)[:n].astype(np.int32) for n in ns]
            live = [r.random(n) < 0.85 for n in ns]
            gn = [np.round(np.exp(r.standard_normal(n)), 2).astype(np.float32) for n in ns]
            rows = [r.standard_normal((n, dims[k])).astype(np.float32) for k, n in enumerate(ns)]
            saving = [r.integers(1, 9, size=ns[0]).astype(np.int32), r.integers(0, 6000, size=ns[1]).astype(np.int32), None]
            budget = [int(r.integers(1, 3000)) if i % 5 else 10 ** 6, None, int(r.integers(1, 200))]
            look = [O.lookup_prune(oc[k], i, ids[k], live[k], None, None, None, 0) for k in range(3)]
            t_ids = [dev(torch, a) if a.size else torch.zeros(1, dtype=torch.int32, device="cuda") for a in ids]
            t_live = [dev(torch, a.astype(np.uint8)) if a.size else torch.zeros(1, dtype=torch.uint8, device="cuda") for a in live]
            t_hit = [dev(torch, look[k]["hit"].astype(np.uint8)) if ns[k] else torch.zeros(1, dtype=torch.uint8, device="cuda") for k in range(3)]
            t_rows = [dev(torch, a) if a.size else torch.zeros((1, dims[k]), device="cuda") for k, a in enumerate(rows)]
            t_gn = [dev(torch, a) if a.size else torch.zeros(1, device="cuda") for a in gn]
            t_sav = [None if a is None else dev(torch, a) for a in saving]
            t_stats = torch.zeros((3, 4), dtype=torch.int64, device="cuda")
            wsb = sum(B.fg_workspace_bytes(B.FG_WS_CACHE_UPDATE, n) for n in ns)
            ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
            B.fg_cache_update_all(cache, i, p, B.update_layers([dict(layer=k + 1, n=ns[k], ids_dev=t_ids[k], live_dev=t_live[k],
                                                                     hit_dev=t_hit[k], gnorm_dev=t_gn[k], h_dev=t_rows[k],
                                                                     h_stride=dims[k] * 4, stats_dev=t_stats[k].data_ptr(),
                                                                     saving_dev=t_sav[k], max_admit=budget[k] or 0)
                                                                for k in range(3)]), ws, wsb, None)
            stats = t_stats.cpu().numpy().tolist()
            for k in range(3):
                st = O.cache_update(oc[k], i, ids[k], live[k], look[k]["hit"], gn[k], p, rows[k], saving=saving[k], budget=budget[k])
                assert stats[k] == [st["admitted"], st["evicted_by_gradient"], st["overwritten"], st["dropped_overflow"]], \
                    f"stats of layer {k + 1} at iteration {i}: {stats[k]} {st}"
                turned_away[k] += st["dropped_overflow"]
                exp = _export(torch, B, cache, caps[k], i + 1, layer=k + 1)
                valid = oc[k].valid_entries(i + 1)
                assert exp["head"] == oc[k].head
                assert dict(zip(exp["nodes"].tolist(), zip(exp["slots"].tolist(), exp["stamps"].tolist()))) == valid
                tab = _tensor_from_ptr(B.fg_cache_table(cache, k + 1), (caps[k], dims[k]), torch.float32, caps[k] * dims[k] * 4,
                                       "cuda").cpu().numpy()
                for v, (s, _) in valid.items():
                    assert np.array_equal(tab[s], oc[k].table[s])
        assert all(t > 0 for t in turned_away), turned_away
    finally:
        B.fg_cache_destroy(cache)


@pytest.mark.parametrize("d_in,d_out,n,n_src,max_deg,relu,seed", [(256, 256, 1024, 6000, 5, False, 0), (64, 64, 256, 1500, 10, True, 1),
                                                                 (128, 96, 700, 700, 3, True, 2), (256, 256, 4000, 9000, 10, True, 3),
                                                                 (24, 40, 50, 90, 4, False, 4), (32, 32, 1, 5, 0, True, 5)])
def test_aggregate_linear_matches_oracle(env, d_in, d_out, n, n_src, max_deg, relu, seed):
    """One call for aggregation + dense update: the one-launch form for small layers, the two-launch form otherwise."""
    torch, B = env
    r = np.random.default_rng(seed)
    deg = r.integers(0, max_deg + 1, size=n)
    start = np.concatenate([[0], np.cumsum(deg)[:-1]]).astype(np.int32)
    end = (start + deg).astype(np.int32)
    col = np.concatenate([r.choice(n_src, size=k, replace=False) for k in deg] + [np.zeros(0, np.int64)]).astype(np.int32)
    rows = np.sort(r.permutation(n)[: max(1, n * 4 // 5)]).astype(np.int32)
    h = r.standard_normal((n_src, d_in)).astype(np.float32)
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    b = (0.1 * r.standard_normal(d_out)).astype(np.float32)
    agg = O.round_to(O.aggregate(start, end, col, rows, h), "f32")
    want = O.round_to(O.linear(h[rows], agg, W, b, relu), "f32")
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    rows_dev[:len(rows)] = dev(torch, rows)
    cnt = dev(torch, np.asarray([len(rows)], dtype=np.int64))
    tcol = dev(torch, col) if len(col) else torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.full((n, d_out), 5.0, dtype=torch.float32, device="cuda")
    ws = torch.zeros((n, d_in), dtype=torch.float32, device="cuda")
    B.fg_aggregate_linear(dev(torch, start), dev(torch, end), tcol, len(col), n, rows_dev, cnt, n, dev(torch, h), n_src, d_in * 4, d_in,
                          d_out, dev(torch, W), dev(torch, b), 1 if relu else 0, ws, d_in * 4, out, n, d_out * 4)
    got = out.cpu().numpy()
    assert T.rel_err_rows(got[rows], want) <= REL_TOL_F32
    assert np.all(got[np.setdiff1d(np.arange(n), rows)] == 5.0)
    one = B.one_launch_layer(n, d_in, d_out)
    assert one == (seed in (0, 1, 2, 5))
    assert bool(ws.any().item()) == (not one)            # the means are stored only by the two-launch form


# ------------------------------------------------------------------------------------------------ backward pass

@pytest.mark.parametrize("n,d", [(1024, 256), (37, 64), (5, 47), (1, 8)])
def test_loss_gradient_and_row_norms_match_oracle(env, n, d):
    torch, B = env
    r = np.random.default_rng(n + d)
    h = (r.standard_normal((n, d)) * 4).astype(np.float32)
    y = r.integers(0, d, size=n).astype(np.int32)
    th, ty = dev(torch, h), dev(torch, y)
    out = torch.zeros((n, d + 4), dtype=torch.float32, device="cuda")        # strided output
    B.fg_softmax_xent_grad(th, d * 4, ty, n, d, out, (d + 4) * 4)
    got = out[:, :d].cpu().numpy()
    assert T.rel_err_rows(got, O.softmax_xent_grad(h, y)) <= REL_TOL_F32
    assert not out[:, d:].any().item()
    norms = torch.zeros(n, dtype=torch.float32, device="cuda")
    B.fg_row_norms(out, (d + 4) * 4, n, d, norms)
    np.testing.assert_allclose(norms.cpu().numpy(), O.row_norms(got).astype(np.float32), rtol=5e-7)


@pytest.mark.parametrize("d_in,d_out,n,n_src,max_deg,relu,seed", [(128, 256, 900, 4000, 9, True, 0), (256, 256, 1500, 1500, 6, True, 1),
                                                                 (64, 64, 300, 700, 5, False, 2), (24, 72, 130, 400, 4, True, 3),
                                                                 (8, 8, 3, 3, 2, True, 4), (256, 256, 1, 40, 30, False, 5)])
def test_layer_backward_matches_oracle(env, d_in, d_out, n, n_src, max_deg, relu, seed):
    """A random block, a random subset of computed rows (the others pruned: end = start), random upstream gradient."""
    torch, B = env
    from fg_inputs.sampler import transpose_block
    r = np.random.default_rng(seed)
    deg = r.integers(0, max_deg + 1, size=n)
    start = np.concatenate([[0], np.cumsum(deg)[:-1]]).astype(np.int32)
    end = (start + deg).astype(np.int32)
    col = np.concatenate([r.choice(n_src, size=k, replace=False) for k in deg] + [np.zeros(0, np.int64)]).astype(np.int32)
    ts, te, tr = transpose_block(start, end, col, n_src)
    live = r.random(n) < 0.9
    hit = live & (r.random(n) < 0.3)
    normal = live & ~hit
    rows = np.flatnonzero(normal).astype(np.int32)
    end_pruned = np.where(normal, end, start).astype(np.int32)
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    dummy = np.zeros((len(rows), d_in))
    want, _, _ = O.layer_backward(start, end_pruned, col, rows, dh, h, dummy, dummy, W, n_src, relu=relu)
    t = lambda a: dev(torch, a) if len(a) else torch.zeros(1, dtype=torch.from_numpy(np.zeros(1, a.dtype)).dtype, device="cuda")
    cnt = dev(torch, np.asarray([len(rows)], dtype=np.int64))
    out = torch.full((n_src, d_in), 7.0, dtype=torch.float32, device="cuda")
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out)
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    norms = torch.full((n_src,), -1.0, dtype=torch.float32, device="cuda")
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    rows_dev[:len(rows)] = dev(torch, rows) if len(rows) else rows_dev[:0]
    B.fg_layer_backward(dev(torch, dh), d_out * 4, dev(torch, h) if relu else None, d_out * 4, n, rows_dev, cnt, n,
                        dev(torch, live.astype(np.uint8)), dev(torch, hit.astype(np.uint8)), dev(torch, start), dev(torch, end_pruned),
                        dev(torch, ts), dev(torch, te), t(tr), len(tr), n_src, d_in, d_out, dev(torch, W), out, d_in * 4, norms, ws, wsb)
    got = out.cpu().numpy()
    np.testing.assert_allclose(norms.cpu().numpy(), O.row_norms(got).astype(np.float32), rtol=5e-7, atol=1e-37)
    e = T.rel_err_rows(got, want)
    assert e <= REL_TOL_F32, f"rel err {e:.3e}"
    assert (np.abs(want).sum(axis=1) == 0).sum() == (np.abs(got).sum(axis=1) == 0).sum()


@pytest.mark.parametrize("kind,d_in,d_out", [("sage", 4, 8), ("sage", 88, 16), ("gcn", 68, 16), ("sage", 256, 64), ("sage", 260, 8), ("gcn", 1024, 8)])
def test_layer_backward_with_hubs_matches_oracle(env, kind, d_in, d_out):
    """Positions on both sides of the number of incoming edges from which a whole workgroup takes one, and of its blocks of
    edges: no edge, 16, 17, 64, 65, 256, 257 and every row, next to each other and far apart; widths of one piece up to rows of
    several passes."""
    torch, B = env
    from fg_inputs.sampler import transpose_block
    r = np.random.default_rng(d_in)
    n, n_src = 700, 1500
    want_deg = {0: 0, 1: n, 2: 257, 3: 17, 4: 16, 700: 256, 701: 65, 702: 64, n_src - 1: 300}
    cols = [[] for _ in range(n)]
    for pos, k in want_deg.items():
        for row in r.choice(n, size=k, replace=False):
            cols[row].append(pos)
    rest = np.setdiff1d(np.arange(n_src), list(want_deg))
    for row in range(n):
        cols[row].extend(r.choice(rest, size=3, replace=False).tolist())
    deg = np.asarray([len(c) for c in cols])
    start = np.concatenate([[0], np.cumsum(deg)[:-1]]).astype(np.int32)
    end, col = (start + deg).astype(np.int32), np.concatenate(cols).astype(np.int32)
    ts, te, tr = transpose_block(start, end, col, n_src)
    assert te[1] - ts[1] == n and te[3] - ts[3] == 17
    hit = r.random(n) < 0.1
    rows = np.flatnonzero(~hit).astype(np.int32)
    end_pruned = np.where(hit, start, end).astype(np.int32)
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    k_w = d_in if kind == "gcn" else 2 * d_in
    W = (r.standard_normal((k_w, d_out)) / np.sqrt(k_w)).astype(np.float32)
    dummy = np.zeros((len(rows), d_in))
    if kind == "gcn":
        want = O.layer_backward_gcn(start, end_pruned, col, rows, dh, h, dummy, W, n_src, relu=True)[0]
    else:
        want = O.layer_backward(start, end_pruned, col, rows, dh, h, dummy, dummy, W, n_src, relu=True)[0]
    cnt = dev(torch, np.asarray([len(rows)], dtype=np.int64))
    out = torch.full((n_src, d_in), 7.0, dtype=torch.float32, device="cuda")
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out, kind=kind)
    ws = torch.full((wsb,), 0xFF, dtype=torch.uint8, device="cuda")      # NaN wherever nothing was computed
    norms = torch.full((n_src,), -1.0, dtype=torch.float32, device="cuda")
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    rows_dev[:len(rows)] = dev(torch, rows)
    B.fg_layer_backward(dev(torch, dh), d_out * 4, dev(torch, h), d_out * 4, n, rows_dev, cnt, n, None, dev(torch, hit.astype(np.uint8)),
                        dev(torch, start), dev(torch, end_pruned), dev(torch, ts), dev(torch, te), dev(torch, tr), len(tr), n_src, d_in,
                        d_out, dev(torch, W), out, d_in * 4, norms, ws, wsb, kind=kind)
    got = out.cpu().numpy()
    np.testing.assert_allclose(norms.cpu().numpy(), O.row_norms(got).astype(np.float32), rtol=5e-7, atol=1e-37)
    # The narrow products sum 8 to 64 terms of about 1 per element, and a hub up to 700 of them with random signs, each rounded
    # to fp32 once: its error is far below 2^-24 times the sum of magnitudes
    scale = np.abs(dh).max() * np.abs(W).sum(axis=1).max()
    tol = np.maximum(REL_TOL_F32 * np.maximum(np.abs(want), np.abs(want).max(axis=1, keepdims=True) / 16), 4 * 2.0 ** -24 * scale)
    assert (np.abs(got - want) <= tol).all(), np.abs(got - want).max()


@pytest.mark.parametrize("kind,d_in,d_out,n,n_src,degrees", [
    ("sage", 256, 16, 300, 333, (20, 24)), ("gcn", 88, 16, 300, 1030, (0, 40)), ("sage", 260, 8, 300, 333, (60, 70)),
    ("sage", 68, 8, 300, 1030, (250, 260)), ("gcn", 1028, 8, 80, 90, (16, 80)), ("sage", 4, 8, 300, 333, (10, 300))])
def test_layer_backward_where_most_positions_are_hubs_matches_oracle(env, kind, d_in, d_out, n, n_src, degrees):
    """Layers whose positions have many incoming edges on average: a hub workgroup holds few positions, several of them hubs,
    taken a wavefront each or (beyond 64 edges, or 256 where there are hubs for every wavefront) by all four."""
    torch, B = env
    from fg_inputs.sampler import transpose_block
    r = np.random.default_rng(d_in + n_src)
    cols = [[] for _ in range(n)]
    for pos in range(n_src):
        for row in r.choice(n, size=min(n, int(r.integers(degrees[0], degrees[1] + 1))), replace=False):
            cols[row].append(pos)
    deg = np.asarray([len(c) for c in cols])
    start = np.concatenate([[0], np.cumsum(deg)[:-1]]).astype(np.int32)
    end, col = (start + deg).astype(np.int32), np.concatenate(cols).astype(np.int32)
    ts, te, tr = transpose_block(start, end, col, n_src)
    rows = np.arange(n, dtype=np.int32)
    dh, h = r.standard_normal((n, d_out)).astype(np.float32), np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    k_w = d_in if kind == "gcn" else 2 * d_in
    W = (r.standard_normal((k_w, d_out)) / np.sqrt(k_w)).astype(np.float32)
    dummy = np.zeros((n, d_in))
    if kind == "gcn":
        want = O.layer_backward_gcn(start, end, col, rows, dh, h, dummy, W, n_src, relu=True)[0]
    else:
        want = O.layer_backward(start, end, col, rows, dh, h, dummy, dummy, W, n_src, relu=True)[0]
    out, norms = torch.full((n_src, d_in), 7.0, device="cuda"), torch.full((n_src,), -1.0, device="cuda")
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out, kind=kind)
    ws = torch.full((wsb,), 0xFF, dtype=torch.uint8, device="cuda")
    B.fg_layer_backward(dev(torch, dh), d_out * 4, dev(torch, h), d_out * 4, n, dev(torch, rows), None, n, None, None, dev(torch, start),
                        dev(torch, end), dev(torch, ts), dev(torch, te), dev(torch, tr), len(tr), n_src, d_in, d_out, dev(torch, W), out,
                        d_in * 4, norms, ws, wsb, kind=kind)
    got = out.cpu().numpy()
    np.testing.assert_allclose(norms.cpu().numpy(), O.row_norms(got).astype(np.float32), rtol=5e-7, atol=1e-37)
    # a product of 8 or 16 terms, rounded once, then sums of up to 300 of them in fp64: as in the test above
    scale = np.abs(dh).max() * np.abs(W).sum(axis=1).max()
    tol = np.maximum(REL_TOL_F32 * np.maximum(np.abs(want), np.abs(want).max(axis=1, keepdims=True) / 16), 4 * 2.0 ** -24 * scale)
    assert (np.abs(got - want) <= tol).all(), np.abs(got - want).max()


@pytest.mark.parametrize("count_on", ["device", "host"])
@pytest.mark.parametrize("d_in,d_out,n,n_rows,relu,seed", [(128, 256, 5000, 4100, True, 0), (256, 256, 700, 700, True, 1),
                                                         (64, 64, 300, 250, False, 2), (24, 72, 130, 77, True, 3),
                                                         (8, 8, 9, 1, True, 4), (128, 256, 40, 0, True, 5),
                                                         (128, 256, 30000, 29001, True, 6), (200, 300, 3000, 2999, True, 7)])
def test_layer_backward_weights_match_oracle(env, d_in, d_out, n, n_rows, relu, seed, count_on):
    """The number of computed rows in device memory, under a bound on the host, or known on the host; the workspace is the one for
    the bound either way."""
    torch, B = env
    r = np.random.default_rng(seed)
    n_src = n + 50
    rows = np.sort(r.permutation(n)[:n_rows]).astype(np.int32)
    h_src = r.standard_normal((n_src, d_in)).astype(np.float32)
    agg = r.standard_normal((n, d_in)).astype(np.float32)        # list order; rows beyond n_rows are never read
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    W = np.zeros((2 * d_in, d_out), dtype=np.float32)
    _, dW, db = O.layer_backward(np.zeros(n, np.int32), np.zeros(n, np.int32), np.zeros(0, np.int32), rows, dh, h, h_src[rows],
                                 agg[:n_rows], W, n_src, relu=relu)
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    if n_rows:
        rows_dev[:n_rows] = dev(torch, rows)
    cnt = dev(torch, np.asarray([n_rows], dtype=np.int64))
    wsb = B.fg_layer_backward_weights_workspace_bytes(n, d_in, d_out)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")           # NaN patterns: every partial must be written
    t_dw = torch.full((2 * d_in, d_out), 3.0, dtype=torch.float32, device="cuda")
    t_db = torch.full((d_out,), 3.0, dtype=torch.float32, device="cuda")
    B.fg_layer_backward_weights(dev(torch, h_src), n_src, d_in * 4, dev(torch, agg), d_in * 4, dev(torch, dh), d_out * 4,
                                dev(torch, h) if relu else None, d_out * 4, n, rows_dev, cnt if count_on == "device" else None,
                                n if count_on == "device" else n_rows, d_in, d_out, t_dw, t_db, ws, wsb)
    e, e_b = T.rel_err_rows(t_dw.cpu().numpy(), dW), T.rel_err_rows(t_db.cpu().numpy()[None, :], db[None, :])
    assert e <= REL_TOL_F32 and e_b <= REL_TOL_F32, f"rel err dW {e:.3e}, db {e_b:.3e}"


@pytest.mark.parametrize("d_in,d_out,n,relu", [
    (64, 64, 300, True), (64, 512, 200, True), (32, 576, 40, False),      # split over K; just beyond what it takes
    (16, 8, 33, True), (40, 72, 700, True), (256, 256, 1500, True), (128, 384, 900, False), (24, 392, 65, True),      # panels of 64, then of 32 columns
    (24, 96, 130, True), (40, 224, 300, False),                            # whole chunks of 32 values, but not pairs of them
    (40, 768, 130, True), (40, 776, 130, True)])                           # the widest, and one that is masked by a launch of its own
@pytest.mark.parametrize("apart", [0, 1])
def test_layer_backward_reads_its_operands_in_place(env, d_in, d_out, n, relu, apart):
    """The input gradient straight from dh, h and W, at the widths where its product changes kernels; `apart`: rows that are one float
    apart and start one float into their memory, so that no 16-byte piece is aligned."""
    torch, B = env
    r = np.random.default_rng(d_out + n)
    n_src = n + 90
    blk = _random_pruned_block(r, n, n_src, 4)
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    dummy = np.zeros((len(blk["rows"]), d_in))
    want, _, _ = O.layer_backward(blk["start"], blk["end"], blk["col"], blk["rows"], dh, h, dummy, dummy, W, n_src, relu=relu)

    def shifted(a, gap):      # (address, bytes per row, the memory)
        mem = torch.full((a.shape[0] * (a.shape[1] + gap) + gap,), float("nan"), device="cuda")
        mem[gap:].view(a.shape[0], a.shape[1] + gap)[:, :a.shape[1]] = dev(torch, a)
        return mem.data_ptr() + 4 * gap, 4 * (a.shape[1] + gap), mem

    t = lambda a: dev(torch, a) if len(a) else torch.zeros(1, dtype=torch.int32, device="cuda")
    (g, g_stride, m0), (a, a_stride, m1) = shifted(dh, apart), shifted(h, apart)
    w_mem = torch.full((W.size + apart,), float("nan"), device="cuda")
    w_mem[apart:] = dev(torch, W.reshape(-1))
    rows = torch.zeros(n, dtype=torch.int32, device="cuda")
    rows[:len(blk["rows"])] = dev(torch, blk["rows"])
    cnt = dev(torch, np.asarray([len(blk["rows"])], dtype=np.int64))
    out, norms = torch.full((n_src, d_in), 7.0, device="cuda"), torch.full((n_src,), -1.0, device="cuda")
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    B.fg_layer_backward(g, g_stride, a if relu else None, a_stride, n, rows, cnt, n, dev(torch, blk["live"].astype(np.uint8)),
                        dev(torch, blk["hit"].astype(np.uint8)), dev(torch, blk["start"]), dev(torch, blk["end"]), dev(torch, blk["ts"]),
                        dev(torch, blk["te"]), t(blk["tr"]), len(blk["tr"]), n_src, d_in, d_out, w_mem.data_ptr() + 4 * apart, out, d_in * 4, norms, ws, wsb)
    e = T.rel_err_rows(out.cpu().numpy(), want)
    assert e <= REL_TOL_F32, f"rel err {e:.3e}"


@pytest.mark.parametrize("d_in,n", [(48, 300), (88, 900)])
@pytest.mark.parametrize("d_out", [32, 72, 96, 160, 224, 288, 352])
def test_layer_backward_of_few_rows_rounds_no_more_than_the_panel_kernel(env, d_in, n, d_out):
    """Input gradient of few rows whose width is no multiple of 64 against 64-bit sums (a block without edges: the product itself). Values of
    the three-way products are rounded when 16 of them are added to the 16 before, and as the result: three times 2^-24 / sqrt(3) of a
    value whose square over its power of two's is 7/3 on average, 3.9e-8 in the 2-norm. A chain of two values at a time would leave 7.5e-8."""
    torch, B = env
    r = np.random.default_rng(d_out + n)
    dh, h = (r.standard_normal((n, d_out)).astype(np.float32) for _ in range(2))
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(d_in)).astype(np.float32)
    zero, flags = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros((2, n), dtype=torch.uint8, device="cuda")
    flags[0] = 1
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out)
    ws, out = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda"), torch.full((n, d_in), 7.0, device="cuda")
    B.fg_layer_backward(dev(torch, dh), d_out * 4, dev(torch, h), d_out * 4, n, torch.arange(n, dtype=torch.int32, device="cuda"), None, n, flags[0], flags[1],
                        zero, zero, zero, zero, zero, 0, n, d_in, d_out, dev(torch, W), out, d_in * 4, None, ws, wsb)
    want = np.where(h > 0, dh, 0).astype(np.float64) @ W[:d_in].astype(np.float64).T
    e = np.linalg.norm(out.cpu().numpy() - want) / np.linalg.norm(want)
    assert e <= 5e-8, f"rel err {e:.2e}"


@pytest.mark.parametrize("kind,layers", [
    ("f32", [(128, 256, 30000, 29001, True), (256, 256, 3000, 2999, True), (256, 64, 300, 250, False)]),       # both tiles, many chunks and few
    ("f32", [(24, 72, 130, 77, True), (72, 8, 40, 0, False)]), ("f32", [(8, 8, 9, 1, False)]),                # one chunk each; an empty layer
    ("bf16", [("f16", 384, 512, 9000, 8000, True), ("bf16", 512, 512, 1024, 1024, True), ("bf16", 512, 64, 100, 90, False)]),
    ("bf16", [("f32", 64, 128, 700, 650, True), ("bf16", 128, 264, 300, 300, False)]), ("bf16", [("bf16", 16, 16, 40, 33, False)] * 8)])
def test_weight_gradients_of_all_layers_in_one_call(env, kind, layers):
    """fg_backward_weights_all against 64-bit sums, layer by layer, with the tolerance of the call for one layer, in the smallest
    workspace that is accepted, filled with NaN patterns: every partial result that is read must have been written."""
    torch, B = env
    r = np.random.default_rng(len(layers))
    bf = kind == "bf16"
    tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
    code = {"f32": B.FG_F32, "f16": B.FG_F16, "bf16": B.FG_BF16}
    act, specs, keep, want = tdt["bf16" if bf else "f32"], [], [], []
    for y in layers:
        src, (d_in, d_out, n, n_rows, relu) = (y[0], y[1:]) if bf else ("f32", y)
        rows = torch.from_numpy(np.sort(r.permutation(n)[:n_rows])).cuda()
        h_src, agg = (torch.randn(m, d_in, device="cuda").to(t) for m, t in ((n + 7, tdt[src]), (n, act)))
        dh, h = torch.randn(n, d_out, device="cuda"), torch.randn(n, d_out, device="cuda").relu().to(act)
        lst, cnt = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.tensor([n_rows], dtype=torch.int64, device="cuda")
        lst[:n_rows] = rows.int()
        dw, db = torch.full((2 * d_in, d_out), 3.0, device="cuda"), torch.full((d_out,), 3.0, device="cuda")
        x = torch.cat([h_src[rows].to(act), agg[:n_rows]], 1).double()
        dz = dh[rows] * (h[rows].float() > 0) if relu else dh[rows]
        want.append((x.t() @ dz.to(act).double(), dz.double().sum(0), dw, db))
        keep.append((h_src, agg, dh, h, lst, cnt))
        specs.append(dict(h_src_dev=h_src, src_stride=d_in * h_src.element_size(), agg_dev=agg, agg_stride=d_in * agg.element_size(), dh_dev=dh,
                          dh_stride=d_out * 4, h_dev=h if relu else None, h_stride=d_out * h.element_size(), rows_dev=lst, n_rows_dev=cnt, max_rows=n,
                          dw_dev=dw, db_dev=db, src_dtype=code[src], n_src=n + 7, n=n, d_in=d_in, d_out=d_out))
    arr = B.weight_grad_layers(specs)
    wsb = B.fg_backward_weights_all_workspace_bytes(B.FG_BF16 if bf else B.FG_F32, arr)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    B.fg_backward_weights_all(B.FG_BF16 if bf else B.FG_F32, arr, ws, wsb)
    for i, (w, b, dw, db) in enumerate(want):
        e, e_b = T.rel_err_rows(dw.cpu().numpy(), w.cpu().numpy()), T.rel_err_rows(db.cpu().numpy()[None], b.cpu().numpy()[None])
        assert e <= REL_TOL_F32 and e_b <= REL_TOL_F32, f"layer {i}: rel err dW {e:.3e}, db {e_b:.3e}"


def _random_pruned_block(r, n, n_src, max_deg):
    """A random block with its transpose, flags, the computed rows and the row ends after pruning."""
    from oracle.sampler_oracle import transpose_block
    deg = r.integers(0, max_deg + 1, size=n)
    start = np.concatenate([[0], np.cumsum(deg)[:-1]]).astype(np.int32)
    end = (start + deg).astype(np.int32)
    col = np.concatenate([r.choice(n_src, size=k, replace=False) for k in deg] + [np.zeros(0, np.int64)]).astype(np.int32)
    ts, te, tr = (np.asarray(x, dtype=np.int32) for x in transpose_block(start, end, col, n_src))
    live = r.random(n) < 0.9
    hit = live & (r.random(n) < 0.3)
    normal = live & ~hit
    return dict(start=start, end=np.where(normal, end, start).astype(np.int32), col=col, ts=ts, te=te, tr=tr, live=live, hit=hit,
                rows=np.flatnonzero(normal).astype(np.int32))


def _call_layer_backward(torch, B, kind, blk, dh, h, W_dev, n, n_src, d_in, d_out, relu):
    t = lambda a: dev(torch, a) if len(a) else torch.zeros(1, dtype=torch.int32, device="cuda")
    rows = blk["rows"]
    cnt = dev(torch, np.asarray([len(rows)], dtype=np.int64))
    out = torch.full((n_src, d_in), 7.0, dtype=torch.float32, device="cuda")
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out, kind=kind)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    norms = torch.full((n_src,), -1.0, dtype=torch.float32, device="cuda")
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    if len(rows):
        rows_dev[:len(rows)] = dev(torch, rows)
    h_dev = None
    if relu:
        h_dev = dev(torch, h).to(torch.bfloat16) if kind == "bf16" else dev(torch, h)
    B.fg_layer_backward(dev(torch, dh), d_out * 4, h_dev, d_out * (2 if kind == "bf16" else 4), n, rows_dev, cnt, n,
                        dev(torch, blk["live"].astype(np.uint8)), dev(torch, blk["hit"].astype(np.uint8)), dev(torch, blk["start"]),
                        dev(torch, blk["end"]), dev(torch, blk["ts"]), dev(torch, blk["te"]), t(blk["tr"]), len(blk["tr"]), n_src, d_in,
                        d_out, W_dev, out, d_in * 4, norms, ws, wsb, kind=kind)
    got = out.cpu().numpy()
    np.testing.assert_allclose(norms.cpu().numpy(), O.row_norms(got).astype(np.float32), rtol=5e-7, atol=1e-37)
    return got


@pytest.mark.parametrize("d_in,d_out,n,n_src,max_deg,relu,seed", [(128, 256, 900, 4000, 9, True, 0), (256, 256, 1500, 1500, 6, True, 1),
                                                                 (64, 64, 300, 700, 5, False, 2), (24, 72, 130, 400, 4, True, 3),
                                                                 (8, 8, 3, 3, 2, True, 4), (256, 256, 1, 40, 30, False, 5)])
def test_layer_backward_gcn_matches_oracle(env, d_in, d_out, n, n_src, max_deg, relu, seed):
    """The GCN layer's input gradient: every computed row hands dm / (deg + 1) to itself and to each sampled neighbour."""
    torch, B = env
    r = np.random.default_rng(100 + seed)
    n_src = max(n_src, n)
    blk = _random_pruned_block(r, n, n_src, max_deg)
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    W = (r.standard_normal((d_in, d_out)) / np.sqrt(d_in)).astype(np.float32)
    want, _, _ = O.layer_backward_gcn(blk["start"], blk["end"], blk["col"], blk["rows"], dh, h, np.zeros((len(blk["rows"]), d_in)), W,
                                      n_src, relu=relu)
    got = _call_layer_backward(torch, B, "gcn", blk, dh, h, dev(torch, W), n, n_src, d_in, d_out, relu)
    e = T.rel_err_rows(got, want)
    assert e <= REL_TOL_F32, f"rel err {e:.3e}"
    assert (np.abs(want).sum(axis=1) == 0).sum() == (np.abs(got).sum(axis=1) == 0).sum()


@pytest.mark.parametrize("d_in,d_out,n,n_src,max_deg,relu,seed", [(128, 256, 900, 4000, 9, True, 0), (256, 256, 1500, 1500, 6, True, 1),
                                                                 (64, 64, 300, 700, 5, False, 2), (24, 80, 130, 400, 4, True, 3),
                                                                 (8, 16, 3, 3, 2, True, 4), (256, 256, 1, 40, 30, False, 5)])
def test_layer_backward_bf16_matches_oracle(env, d_in, d_out, n, n_src, max_deg, relu, seed):
    """Mixed precision: dz and W enter dz . W^T as bf16; the oracle rounds the same way and multiplies in fp64, so what is
    left is the device's fp32 summation."""
    torch, B = env
    r = np.random.default_rng(200 + seed)
    n_src = max(n_src, n)
    blk = _random_pruned_block(r, n, n_src, max_deg)
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = O.round_bf16(np.maximum(r.standard_normal((n, d_out)), 0))
    W = O.round_bf16(r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in))
    dummy = np.zeros((len(blk["rows"]), d_in))
    want, _, _ = O.layer_backward(blk["start"], blk["end"], blk["col"], blk["rows"], dh, h, dummy, dummy, W, n_src, relu=relu,
                                  compute_dtype="bf16")
    got = _call_layer_backward(torch, B, "bf16", blk, dh, h, dev(torch, W).to(torch.bfloat16), n, n_src, d_in, d_out, relu)
    e = T.rel_err_rows(got, want)
    print(f"layer backward bf16 {d_in}x{d_out}: rel err {e:.3e}")
    assert e <= REL_TOL_F32, f"rel err {e:.3e}"
    # against the unrounded product the difference is of bf16 size: the rounding really happens on the device
    plain, _, _ = O.layer_backward(blk["start"], blk["end"], blk["col"], blk["rows"], dh, h, dummy, dummy, W, n_src, relu=relu)
    if len(blk["rows"]) > 10:
        assert T.rel_err_rows(got, plain) > 1e-4


@pytest.mark.parametrize("src,d_in,d_out,n,n_rows,relu,seed", [("bf16", 128, 256, 5000, 4100, True, 0), ("f16", 256, 256, 700, 700, True, 1),
                                                             ("f32", 64, 64, 300, 250, False, 2), ("bf16", 24, 72, 130, 77, True, 3),
                                                             ("f16", 8, 8, 9, 1, True, 4), ("bf16", 128, 256, 40, 0, True, 5),
                                                             ("f16", 384, 256, 2000, 1900, True, 6)])
def test_layer_backward_weights_bf16_match_oracle(env, src, d_in, d_out, n, n_rows, relu, seed):
    """Mixed precision: [h_src ‖ agg] and dz enter the product as bf16, the bias gradient sums the unrounded dz."""
    torch, B = env
    r = np.random.default_rng(300 + seed)
    n_src = n + 50
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
    code = {"f16": B.FG_F16, "bf16": B.FG_BF16, "f32": B.FG_F32}
    rows = np.sort(r.permutation(n)[:n_rows]).astype(np.int32)
    h_src = O.round_to(r.standard_normal((n_src, d_in)), src).astype(np.float32)
    agg = O.round_bf16(r.standard_normal((n, d_in)))
    dh = r.standard_normal((n, d_out)).astype(np.float32)
    h = O.round_bf16(np.maximum(r.standard_normal((n, d_out)), 0))
    W = np.zeros((2 * d_in, d_out), dtype=np.float32)
    none = np.zeros(n, np.int32)
    _, dW, db = O.layer_backward(none, none, np.zeros(0, np.int32), rows, dh, h, O.round_bf16(h_src[rows].astype(np.float64)), agg[:n_rows],
                                 W, n_src, relu=relu, compute_dtype="bf16")
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    if n_rows:
        rows_dev[:n_rows] = dev(torch, rows)
    cnt = dev(torch, np.asarray([n_rows], dtype=np.int64))
    wsb = B.fg_layer_backward_weights_bf16_workspace_bytes(n, d_in, d_out)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")           # NaN patterns: whatever is read must have been written
    t_dw = torch.full((2 * d_in, d_out), 3.0, dtype=torch.float32, device="cuda")
    t_db = torch.full((d_out,), 3.0, dtype=torch.float32, device="cuda")
    ssz = 4 if src == "f32" else 2
    B.fg_layer_backward_weights_bf16(dev(torch, h_src).to(tdt[src]), n_src, d_in * ssz, code[src], dev(torch, agg).to(torch.bfloat16),
                                     d_in * 2, dev(torch, dh), d_out * 4, dev(torch, h).to(torch.bfloat16) if relu else None, d_out * 2,
                                     n, rows_dev, cnt, n, d_in, d_out, t_dw, t_db, ws, wsb)
    e, e_b = T.rel_err_rows(t_dw.cpu().numpy(), dW), T.rel_err_rows(t_db.cpu().numpy()[None, :], db[None, :])
    print(f"weight gradients bf16 {src} {d_in}x{d_out}: rel err dW {e:.3e}, db {e_b:.3e}")
    assert e <= REL_TOL_F32 and e_b <= REL_TOL_F32, f"rel err dW {e:.3e}, db {e_b:.3e}"


@pytest.mark.parametrize("n,d", [(3, 256), (1031, 257), (5000, 260), (2, 1024), (9, 1025), (4, 2600), (1536, 300), (1537, 300),
                                 (1600, 512), (1600, 513), (1600, 640), (1600, 641), (4100, 700)])
def test_loss_gradient_of_wide_rows(env, n, d):
    """Rows of one wavefront and of four, within and beyond what their registers keep; more rows than workgroups."""
    torch, B = env
    r = np.random.default_rng(n + d)
    h = (r.standard_normal((n, d)) * 4).astype(np.float32)
    y = r.integers(0, d, size=n).astype(np.int32)
    out = torch.zeros((n, d + 4), dtype=torch.float32, device="cuda")
    B.fg_softmax_xent_grad(dev(torch, h), d * 4, dev(torch, y), n, d, out, (d + 4) * 4)
    assert T.rel_err_rows(out[:, :d].cpu().numpy(), O.softmax_xent_grad(h, y)) <= REL_TOL_F32
    assert not out[:, d:].any().item()


@pytest.mark.parametrize("kind", ["sage", "bf16"])
@pytest.mark.parametrize("d_out,pad", [(16, 0), (16, 4), (272, 1), (272, 0)])
def test_layer_backward_strides(env, kind, d_out, pad):
    """The mask four columns at a time and one at a time (rows of dh and h padded off 16 bytes) give the same gradient."""
    torch, B = env
    r = np.random.default_rng(d_out + pad)
    n, n_src, d_in = 130, 300, 24
    blk = _random_pruned_block(r, n, n_src, 5)
    dh, h = r.standard_normal((n, d_out)).astype(np.float32), np.maximum(r.standard_normal((n, d_out)), 0).astype(np.float32)
    W = (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)
    act = torch.bfloat16 if kind == "bf16" else torch.float32
    rows = torch.zeros(n, dtype=torch.int32, device="cuda")
    rows[:len(blk["rows"])] = dev(torch, blk["rows"])
    cnt = dev(torch, np.asarray([len(blk["rows"])], dtype=np.int64))
    wsb = B.fg_layer_backward_workspace_bytes(n, n, d_in, d_out, kind=kind)
    got = []
    for p in (0, pad):
        wide = lambda a, dt: torch.nn.functional.pad(dev(torch, a), (0, p), value=float("nan")).to(dt).contiguous()
        tdh, th = wide(dh, torch.float32), wide(h, act)
        out, norms = torch.full((n_src, d_in), 7.0, device="cuda"), torch.full((n_src,), -1.0, device="cuda")
        ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
        B.fg_layer_backward(tdh, (d_out + p) * 4, th, (d_out + p) * th.element_size(), n, rows, cnt, n, dev(torch, blk["live"].astype(np.uint8)),
                            dev(torch, blk["hit"].astype(np.uint8)), dev(torch, blk["start"]), dev(torch, blk["end"]), dev(torch, blk["ts"]),
                            dev(torch, blk["te"]), dev(torch, blk["tr"]), len(blk["tr"]), n_src, d_in, d_out, dev(torch, W).to(act), out,
                            d_in * 4, norms, ws, wsb, kind=kind)
        got.append((out.cpu().numpy(), norms.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("kind,src,d_in,d_out,n,n_rows,rows,relu", [
    ("f32", "f32", 68, 132, 32768, 32767, "list", True),          # 256 x 128 tiles, halves padded to 128 columns
    ("f32", "f32", 128, 64, 33000, 100, "list", False),            # most chunks without a row
    ("f32", "f32", 64, 128, 33000, 33000, "all", True),            # many rows, one tile of 128
    ("f32", "f32", 60, 36, 2049, 2000, "bad", True), ("f32", "f32", 132, 260, 300, 33, "bad", False),
    ("bf16", "f16", 136, 264, 12000, 11111, "list", True),         # 256 x 256 tiles, ragged in both directions
    ("bf16", "bf16", 136, 264, 12000, 12000, "all", False), ("bf16", "f32", 136, 264, 12000, 65, "bad", True),
    ("bf16", "f16", 520, 136, 5500, 5400, "bad", True), ("bf16", "f32", 72, 40, 1000, 999, "bad", True),
    ("f32", "f32", 64, 64, 500, 480, "short", True), ("bf16", "bf16", 64, 64, 500, 480, "short", True),
    ("f32", "f32", 1024, 1020, 96, 95, "bad", True), ("bf16", "bf16", 1024, 1032, 300, 290, "list", True),      # one chunk
    ("bf16", "f16", 520, 1024, 1500, 33, "short", True), ("f32", "f32", 36, 52, 5, 3, "list", False)])
def test_weight_gradients_tiles_and_chunks(env, kind, src, d_in, d_out, n, n_rows, rows, relu):
    """Both tile sizes of the weight gradients, at sizes that no tile, chunk or step divides; lists that name every position
    ("all": no list at all), some, positions that do not exist ("bad": they contribute nothing) and positions without own
    features ("short": left out of the fp32 product, zeros in the mixed one), in a workspace that holds NaN patterns. Reference: torch in fp64 on the operands as the product takes them."""
    torch, B = env
    g = torch.Generator(device="cuda").manual_seed(n + d_in)
    bf = kind == "bf16"
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
    code = {"f16": B.FG_F16, "bf16": B.FG_BF16, "f32": B.FG_F32}
    act_t = torch.bfloat16 if bf else torch.float32
    n_src = n - 40 if rows == "short" else n + 7
    rnd = lambda *shape: torch.randn(*shape, device="cuda", generator=g)
    h_src, agg, dh, h = rnd(n_src, d_in).to(tdt[src]), rnd(n, d_in).to(act_t), rnd(n, d_out), rnd(n, d_out).to(act_t)
    pos = torch.arange(n, device="cuda") if rows == "all" else torch.sort(torch.randperm(n, device="cuda", generator=g)[:n_rows])[0]
    lst = torch.zeros(n, dtype=torch.int32, device="cuda")
    lst[:n_rows] = pos.int()
    good = torch.ones(n_rows, dtype=torch.bool, device="cuda")
    if rows == "bad":
        good[::5] = False
        lst[:n_rows][~good] = torch.tensor([-1, n, n_src + 3], dtype=torch.int32, device="cuda").repeat(n_rows)[:int((~good).sum())]
    if rows == "short" and not bf:
        good = pos < n_src
    own = torch.where((pos < n_src)[:, None], h_src[pos.clamp(max=n_src - 1)], torch.zeros_like(h_src[:1]))
    x = torch.cat([own.to(torch.bfloat16) if bf else own, agg[:n_rows]], 1)
    dz = torch.where(h[pos] > 0, dh[pos], torch.zeros_like(dh[pos])) if relu else dh[pos]
    x, dz = x[good], dz[good]
    want = x.double().t() @ (dz.to(torch.bfloat16) if bf else dz).double()
    want_b = dz.double().sum(0)
    cnt = dev(torch, np.asarray([n_rows], dtype=np.int64))
    size = B.fg_layer_backward_weights_bf16_workspace_bytes if bf else B.fg_layer_backward_weights_workspace_bytes
    wsb = size(n, d_in, d_out)
    assert all(size(m, d_in, d_out) <= wsb for m in (0, 1, 32, 64, n // 2, n - 1))      # a workspace serves fewer rows too
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    dw, db = torch.full((2 * d_in, d_out), 3.0, device="cuda"), torch.full((d_out,), 3.0, device="cuda")
    lst_arg, act_arg, asz = None if rows == "all" else lst, h if relu else None, 2 if bf else 4
    if bf:
        B.fg_layer_backward_weights_bf16(h_src, n_src, d_in * h_src.element_size(), code[src], agg, d_in * 2, dh, d_out * 4, act_arg,
                                         d_out * asz, n, lst_arg, cnt, n, d_in, d_out, dw, db, ws, wsb)
    else:
        B.fg_layer_backward_weights(h_src, n_src, d_in * 4, agg, d_in * 4, dh, d_out * 4, act_arg, d_out * asz, n, lst_arg, cnt, n,
                                    d_in, d_out, dw, db, ws, wsb)
    e, e_b = float((dw.double() - want).norm() / want.norm()), float((db.double() - want_b).norm() / want_b.norm())
    # the chunks of these shapes have at most 512 rows, summed in fp32 steps of 16: at most 32 roundings of half an ulp each, of
    # sums that grow to the size of the chunk's result; the bias sums are fp64 over fp32 sums of eight
    assert e <= 32 * 2.0 ** -24 and e_b <= 8 * 2.0 ** -24, f"rel err dW {e:.3e}, db {e_b:.3e}"


@pytest.mark.parametrize("d_in,d_out,n", [(1024, 1024, 9000), (512, 512, 33000), (256, 1020, 70000), (64, 512, 66000)])
def test_weight_gradients_of_long_chunks(env, d_in, d_out, n):
    """fp32, wide results over many rows of all-positive operands, where the roundings of a running sum add up: chunks of up to
    4096 rows."""
    torch, B = env
    g = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *shape: torch.rand(*shape, device="cuda", generator=g)
    h_src, agg, dh, h = rnd(n, d_in), rnd(n, d_in), rnd(n, d_out), torch.randn(n, d_out, device="cuda", generator=g)
    cnt = dev(torch, np.asarray([n], dtype=np.int64))
    wsb = B.fg_layer_backward_weights_workspace_bytes(n, d_in, d_out)
    assert wsb >= -(-n // 4096) * 2 * d_in * d_out * 4      # a partial result for every 4096 rows
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    dw, db = torch.full((2 * d_in, d_out), 3.0, device="cuda"), torch.full((d_out,), 3.0, device="cuda")
    B.fg_layer_backward_weights(h_src, n, d_in * 4, agg, d_in * 4, dh, d_out * 4, h, d_out * 4, n, None, cnt, n, d_in, d_out, dw, db, ws, wsb)
    want = torch.zeros((2 * d_in, d_out), dtype=torch.float64, device="cuda")
    dz = torch.where(h > 0, dh, torch.zeros_like(dh))
    for k in range(0, n, 8192):
        want += torch.cat([h_src[k:k + 8192], agg[k:k + 8192]], 1).double().t().contiguous() @ dz[k:k + 8192].double()
    e, e_b = float((dw.double() - want).norm() / want.norm()), float((db.double() - dz.double().sum(0)).norm() / dz.double().sum(0).norm())
    # a chunk's sum grows by 256 steps of 16 rows, each rounded once: sqrt(256) half-ulps if the roundings are independent
    assert e <= 16 * 2.0 ** -24 and e_b <= 8 * 2.0 ** -24, f"rel err dW {e:.3e}, db {e_b:.3e}"


@pytest.mark.parametrize("kind,d_in,d_out", [("f32", 68, 132), ("bf16", 136, 264)])
def test_weight_gradients_of_operands_beyond_4_gb(env, kind, d_in, d_out):
    """Rows 128 MB apart, the last ones beyond 2^32 bytes from the first: the same bits as from rows close together, with and
    without a bias gradient."""
    torch, B = env
    n, stride, bf = 40, 1 << 27, kind == "bf16"
    far = torch.empty(n * stride, dtype=torch.uint8, device="cuda")
    r = np.random.default_rng(d_in)
    lst, cnt = dev(torch, np.sort(r.permutation(n)[:37]).astype(np.int32)), dev(torch, np.asarray([37], dtype=np.int64))
    at, near, wide = 0, [], []
    for cols, dt in ((d_in, torch.bfloat16 if bf else torch.float32), (d_in, torch.bfloat16 if bf else torch.float32), (d_out, torch.float32),
                     (d_out, torch.bfloat16 if bf else torch.float32)):
        a = dev(torch, r.standard_normal((n, cols)).astype(np.float32)).to(dt)
        size = cols * a.element_size()
        view = far.view(n, stride)[:, at:at + size]
        view.copy_(a.view(torch.uint8))
        near.append((a, size))
        wide.append((view, stride))
        at += 4096
    size = B.fg_layer_backward_weights_bf16_workspace_bytes if bf else B.fg_layer_backward_weights_workspace_bytes
    wsb = size(n, d_in, d_out)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")
    got = []
    for (h_src, agg, dh, h), bias in ((near, True), (wide, True), (wide, False)):
        dw, db = torch.full((2 * d_in, d_out), 3.0, device="cuda"), torch.full((d_out,), 3.0, device="cuda")
        tail = (agg[0].data_ptr(), agg[1], dh[0].data_ptr(), dh[1], h[0].data_ptr(), h[1], n, lst, cnt, n, d_in, d_out, dw, db if bias else None, ws, wsb)
        if bf:
            B.fg_layer_backward_weights_bf16(h_src[0].data_ptr(), n, h_src[1], B.FG_BF16, *tail)
        else:
            B.fg_layer_backward_weights(h_src[0].data_ptr(), n, h_src[1], *tail)
        got.append((dw.cpu().numpy(), db.cpu().numpy()))
    pos = lst.cpu().long()
    x = torch.cat([near[0][0].cpu()[pos].double(), near[1][0].cpu()[:37].double()], 1)
    dz = torch.where(near[3][0].cpu()[pos] > 0, near[2][0].cpu()[pos], torch.zeros(1))
    want = x.t() @ (dz.to(torch.bfloat16) if bf else dz).double()
    assert np.linalg.norm(got[0][0] - want.numpy()) <= 32 * 2.0 ** -24 * np.linalg.norm(want.numpy())
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert np.array_equal(got[0][0], got[2][0]) and (got[2][1] == 3.0).all()


def test_iterations_gcn_layers_with_backward_pass(env):
    """GCN layers with the gradient norms from the backward pass (input and weight gradients of every layer)."""
    torch, B = env
    import dataclasses
    hits, _ = run_workload_parity(torch, wl.WORKLOADS["tiny"], 12, model="gcn", backward=True)
    assert hits > 50
    assert run_workload_parity(torch, wl.WORKLOADS["tiny"], 6, model="gcn", backward=True, fused=True)[0] > 0
    w3 = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                             train_nodes=20_000, cache_capacity=20_000, t_stale=6)
    assert run_workload_parity(torch, w3, 8, p_grad=0.7, model="gcn", backward=True, fused=True)[0] > 0
    # half of the input columns fit one tile of the weight gradients, all of them do not
    w4 = dataclasses.replace(w3, feat_dim=104, hidden=72, num_nodes=30_000, num_edges=500_000, batch=256, train_nodes=None)
    assert run_workload_parity(torch, w4, 4, p_grad=0.7, model="gcn", backward=True, fused=True, device_sampler=True, device_counts=True)[0] > 0


def test_iterations_bf16_with_backward_pass(env):
    """The mixed-precision model with the gradient norms from its backward pass: a small three-layer workload with fp16
    features and bf16 embeddings, weights and cache."""
    torch, B = env
    import dataclasses
    w = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small-bf16", num_nodes=200_000, num_edges=4_000_000, batch=128,
                            train_nodes=20_000, cache_capacity=20_000, t_stale=6, feat_dtype="f16", compute_dtype="bf16")
    assert run_workload_parity(torch, w, 8, p_grad=0.7, backward=True, fused=True)[0] > 0
    assert run_workload_parity(torch, w, 5, p_grad=0.7, backward=True)[0] > 0


def test_iterations_very_large_bf16_with_backward_pass(env):
    """The paper-scale mixed-precision workload (nodes divided by 8 as in the forward test) with real gradient norms."""
    torch, B = env
    w = wl.WORKLOADS["very_large"].scaled(8)
    hits, worst = run_workload_parity(torch, w, 4, check_numeric_every=3, sample_rows=20000, fused=True, col_ids=True, backward=True)
    assert hits > 0


def test_iterations_tiny_with_backward_pass(env):
    """Whole iterations whose gradient norms come from the backward pass (loss, layer backward, row norms)."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    hits, worst = run_workload_parity(torch, w, 12, backward=True)
    assert hits > 50
    hits, worst = run_workload_parity(torch, w, 6, backward=True, fused=True)
    assert hits > 0


def test_iterations_three_layers_with_backward_pass(env):
    torch, B = env
    import dataclasses
    w = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                            train_nodes=20_000, cache_capacity=20_000, t_stale=6)
    hits, worst = run_workload_parity(torch, w, 10, p_grad=0.7, backward=True, fused=True)
    assert hits > 0


def test_iterations_large_hbm_full_size_with_backward_pass(env):
    """The benchmarked workload at full size with real gradient norms (the configuration bench.py --backward times)."""
    torch, B = env
    w = wl.WORKLOADS["large_hbm"]
    hits, worst = run_workload_parity(torch, w, 4, check_numeric_every=3, sample_rows=20000, fused=True, backward=True)
    assert hits > 0


# ------------------------------------------------------------------------------------------------ whole iterations

def run_workload_parity(torch, w, iterations, check_numeric_every=1, t_stale=None, p_grad=None, capacity=None,
                        sample_rows=None, feat_table=None, fused=False, one_launch_top_down=True, feature_side=None,
                        backward=False, stabilization=0, model="sage", conditioned=False, col_ids=False,
                        fetch_with_loader=True, admit_budget=None, device_sampler=False, overlap_update=True,
                        lookahead=False, device_counts=False, fuse_small_layers=False, copy_own_rows=False):
    """Run `iterations` iterations on both sides from an empty cache; compare everything after every call sequence.

    copy_own_rows: the loader copies the layer-1 nodes' own feature rows out for the dense update (compared bit for bit
    here); otherwise, where the pipeline can, that update reads them from the table itself and no copy exists to compare.

    feature_side = dict(n_hot, buffer_bytes[, poison]): both sides share the cache's buffer with the raw features of the
    graph's n_hot hottest nodes (Section 4.2). poison: once the rows are placed, the table rows of those nodes are
    negated on both sides, so a row read from the wrong place shows.
    conditioned: for narrow layers. The bar is 1e-5 of max(|ref|, rowmax/16); where a row's largest output is small next to
    the terms it is summed from, one fp32 rounding of those terms already exceeds that, whatever the kernel. The bound
    used is then max(1e-5, 4 fp32 half-ulps of sum |terms| over the same denominator), computed from the oracle's values.
    device_counts (with device_sampler): the sampled mini-batch is run with its layer sizes still in device memory (bounds on
    the host); they are read back, and the sample compared with the oracle's, only after the iteration has been launched.
    backward: the gradient norms come from the backward pass of a softmax cross-entropy loss on the seeds' synthetic
    labels. The embedding gradients and their norms are compared within tolerance; the admission decisions are then taken
    on both sides from the device's norms (the same fp32 values), so that cache state stays comparable bit for bit.
    """
    g = wl.make_graph(w)
    frows = G.feature_accessor(w)
    fs = feature_side
    hot = g.hottest(fs["n_hot"]) if fs else None
    hp, weights, feat_table = G.make_hotpath(w, feat_table=feat_table, t_stale=t_stale, p_grad=p_grad, capacity=capacity,
                                             fused_input=fused, one_launch_top_down=one_launch_top_down,
                                             update_all=one_launch_top_down, hot_ids=hot,
                                             buffer_bytes=fs["buffer_bytes"] if fs else None, backward=backward, weight_grads=backward, stabilization=stabilization, model=model,
                                             fetch_with_loader=fetch_with_loader, admit_budget=admit_budget,
                                             overlap_update=overlap_update, fuse_small_layers=fuse_small_layers,
                                             copy_own_rows=copy_own_rows)
    from paper_2301_07482_amd import binding as FGB
    bc = None
    if fs:
        bc = G.make_oracle_bidirectional(w, fs["buffer_bytes"], capacity=capacity, t_stale=t_stale)
        bc.fill_features(hot, frows, w.feat_dtype)
        caches = bc.rings
        assert hp.feature_side and FGB.fg_cache_feature_rows(hp.cache) == len(hot)
        assert [FGB.fg_cache_ring_offset(hp.cache, l) for l in bc.rings] == [bc.ring_base[l] for l in bc.rings]
        if fs.get("poison"):
            torch.cuda.synchronize()
            feat_table[torch.as_tensor(hot.astype(np.int64), device=feat_table.device)] *= -1
            clean, hot_set = frows, set(hot.tolist())

            def frows(ids):
                rows = clean(ids)
                flip = np.asarray([int(v) in hot_set for v in np.asarray(ids).tolist()], dtype=bool)
                rows[flip] = -rows[flip]
                return rows
    else:
        caches = G.make_oracle_caches(w, capacity=capacity, t_stale=t_stale)
    from paper_2301_07482_amd.pipeline import DeviceBatch
    served = 0
    dims = wl.layer_dims(w)
    L = w.num_layers
    p = w.p_grad if p_grad is None else p_grad
    total_hits = 0
    worst = worst_e2e = worst_bw = worst_w = 0.0
    sampler = None
    if device_sampler:      # the graph written out as a CSR on the device; the oracle samples from a copy of the same CSR
        from fg_inputs import device as fdev, rng
        from fg_inputs.sampler import MiniBatch
        from oracle import sampler_oracle as S
        from paper_2301_07482_amd.pipeline import DeviceSampler
        indptr_t, indices_t = fdev.chunglu_csr(g)
        csr = (indptr_t.cpu().numpy(), indices_t.cpu().numpy())
        sampler = DeviceSampler(indptr_t, indices_t, w.num_nodes, w.fanouts, w.batch, transposes=backward)
    try:
        def prepare(it):
            """Mini-batch `it` on both sides: sampled (or sampled on the device and compared), uploaded, with its norms."""
            if sampler is not None:
                seeds = wl.seed_nodes(w, it)
                key = int(rng.make_key(w.seed, 0x5A3, it))
                o = S.sample_minibatch(csr[0], csr[1], seeds, w.fanouts, key)
                a32 = lambda x: np.asarray(x, dtype=np.int32)
                mb = MiniBatch(L, [a32(x) for x in o["ids"]], [None] + [a32(x) for x in o["start"][1:]],
                               [None] + [a32(x) for x in o["end"][1:]], [None] + [a32(x) for x in o["col"][1:]])
                bt = sampler.sample(dev(torch, seeds.astype(np.int32)), key, finish=not device_counts)

                want_t = {}
                if backward:      # the transposes of the blocks as sampled (the iteration prunes mb's row ends in place)
                    from oracle import sampler_oracle as SO
                    want_t = {l: SO.transpose_block(mb.start[l], mb.end[l], mb.col[l], len(mb.ids[l - 1])) for l in range(2, L + 1)}

                def verify(bt=bt, mb=mb, o=o, it=it, want_t=want_t):
                    """The device's sample against the oracle's (layer sizes read back first, if they were not yet)."""
                    if bt.n_dev[0] is not None:
                        bt.finish()
                    assert bt.n == [len(x) for x in mb.ids] and bt.nnz[1:] == [len(mb.col[l]) for l in range(1, L + 1)]
                    for l in range(L + 1):
                        assert np.array_equal(bt.ids[l].cpu().numpy()[:bt.n[l]], mb.ids[l]), f"sampled nodes, iteration {it} layer {l}"
                    for l in range(1, L + 1):
                        assert np.array_equal(bt.start[l].cpu().numpy()[:bt.n[l]], mb.start[l])
                        assert np.array_equal(bt.col[l].cpu().numpy()[:bt.nnz[l]], mb.col[l]), f"sampled block, iteration {it} layer {l}"
                    assert np.array_equal(bt.col_ids1.cpu().numpy()[:bt.nnz[1]], a32(o["col_ids"][1]))
                    if backward:
                        for l in range(2, L + 1):      # the device's transposed blocks against the oracle's definition
                            ts, te, tr = want_t[l]
                            assert bt.t_start[l].cpu().numpy()[:bt.n[l - 1]].tolist() == ts and bt.t_end[l].cpu().numpy()[:bt.n[l - 1]].tolist() == te
                            assert bt.t_row[l].cpu().numpy()[:bt.nnz[l]].tolist() == tr, f"transposed block, iteration {it} layer {l}"

                if device_counts:      # the sizes stay on the device until the iteration has run; the row ends are pruned by then
                    bt.verify_sample = verify
                else:
                    for l in range(1, L + 1):
                        assert np.array_equal(bt.end[l].cpu().numpy()[:bt.n[l]], mb.end[l])
                    verify()
                gn = {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)}
                bt.gnorm = {l: dev(torch, x) for l, x in gn.items()}
                labels = None
                if backward:
                    labels = wl.node_labels(w, mb.ids[L])
                    bt.labels = dev(torch, labels.astype(np.int32))
            else:
                mb = wl.minibatch(w, g, it)
                gn = {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)}
                labels = wl.node_labels(w, mb.ids[L]) if backward else None
                bt = DeviceBatch(mb, None if backward else gn, labels=labels, col_ids=col_ids)   # uploaded before the oracle prunes its copy
            return mb, bt, gn, labels

        ahead = prepare(0) if (lookahead and iterations) else None
        for it in range(iterations):
            mb, bt, gn, labels = ahead if lookahead else prepare(it)
            ahead = prepare(it + 1) if (lookahead and it + 1 < iterations) else None     # uploaded before this iteration runs
            if bc is not None:
                # what the loader is about to find on the feature side, for every node of the input layer (or a sample)
                n0 = len(mb.ids[0])
                pick = np.arange(n0) if sample_rows is None or n0 <= sample_rows else np.sort(
                    np.random.default_rng(1000 + it).choice(n0, sample_rows, replace=False))
                ranks, found = hp.feature_ranks(bt.ids[0], n0)
                assert np.array_equal(ranks[pick], np.asarray([bc.feature_rank(int(v)) for v in mb.ids[0][pick]], dtype=np.int32)), \
                    f"feature-side ranks, iteration {it}"
                assert found == int((ranks >= 0).sum())
            rec = O.iteration(mb, it, caches, frows, weights, gn, p, dims, w.feat_dtype, w.compute_dtype, feature_side=bc,
                              labels=labels, update=not backward, stabilization=stabilization, model=model,
                              admit_budget=admit_budget)
            served += int(rec["feature_from_buffer"].sum())
            # device cache rows at the slots about to be hit, read before this iteration's update recycles slots
            pre_rows = {l: hp.cache_rows(l, rec["look"][l]["hit_slot"]) for l in range(1, L) if len(rec["look"][l]["hit_pos"])}
            hp.run(bt, it, next_bt=ahead[1] if ahead is not None else None)
            if getattr(bt, "verify_sample", None) is not None:
                bt.verify_sample()
            snap = hp.snapshot(bt)
            if backward:
                # (a) every call against the oracle on the SAME inputs (the device's own H and dH of the layer above), so
                #     that a ReLU output that is +0 on one side and a rounding error above it on the other cannot matter
                bw = rec["backward"]
                nl = [len(x) for x in mb.ids]
                dHd = {l: hp.dH[l][:nl[l]].cpu().numpy() for l in range(1, L + 1)}
                Hd = {l: G.to_f32(hp.H[l][:nl[l]]) for l in range(1, L + 1)}
                e = T.rel_err_rows(dHd[L], O.softmax_xent_grad(Hd[L], labels))
                assert e <= REL_TOL_F32, f"loss gradient, iteration {it}: rel err {e:.3e}"
                cd = w.compute_dtype
                tol_bw = REL_TOL_F32 if cd == "f32" else 2e-5     # bf16 operands: exact products, fp32 sums on both sides of the bar
                for l in range(L, 1, -1):
                    rows = rec["look"][l]["normal_pos"]
                    if model == "gcn":
                        want, _, _ = O.layer_backward_gcn(mb.start[l], mb.end[l], mb.col[l], rows, dHd[l], Hd[l],
                                                          np.zeros((len(rows), dims[l - 1])), weights[l][0], nl[l - 1], relu=(l < L))
                    else:
                        dummy = np.zeros((len(rows), dims[l - 1]))
                        want, _, _ = O.layer_backward(mb.start[l], mb.end[l], mb.col[l], rows, dHd[l], Hd[l], dummy, dummy, weights[l][0],
                                                      nl[l - 1], relu=(l < L), compute_dtype=cd)
                    e = T.rel_err_rows(dHd[l - 1], want)
                    worst_bw = max(worst_bw, e)
                    assert e <= tol_bw, f"dH[{l - 1}] iteration {it} (same inputs): rel err {e:.3e}"
                # weight gradients, on the device's own inputs of each layer (fused loader: the neighbours' rows of the input
                # layer were never materialised, the oracle's bit-identical feature rows take their place)
                for l in range(L, 0, -1):
                    rows = rec["look"][l]["normal_pos"]
                    if model == "gcn":      # the propagated rows as the device left them: by-position half ‖ list-order half
                        hw = dims[l - 1] // 2
                        idx = torch.as_tensor(rows.astype(np.int64), device="cuda")
                        m_dev = np.concatenate([G.to_f32(hp.MEANPOS_l[l][: bt.n[l] * hw].view(bt.n[l], hw)[idx]),
                                                G.to_f32(hp.AGG_l[l][: len(rows) * hw].view(len(rows), hw))], axis=1)
                        _, dW, db = O.layer_backward_gcn(mb.start[l], mb.end[l], mb.col[l], rows, dHd[l], Hd[l], m_dev, weights[l][0],
                                                         nl[l - 1], relu=(l < L))
                    else:
                        h_prev = rec["H"][0].astype(np.float32) if (fused and l == 1) else G.to_f32(hp.H[l - 1][:nl[l - 1]])
                        h_self = h_prev[rows] if cd == "f32" else O.round_bf16(h_prev[rows].astype(np.float64))
                        agg_dev = G.to_f32(hp.AGG_l[l][: len(rows) * dims[l - 1]].view(len(rows), dims[l - 1]))
                        _, dW, db = O.layer_backward(mb.start[l], mb.end[l], mb.col[l], rows, dHd[l], Hd[l], h_self, agg_dev,
                                                     weights[l][0], nl[l - 1], relu=(l < L), compute_dtype=cd)
                    e = T.rel_err_rows(hp.dW[l].cpu().numpy(), dW)
                    e_b = T.rel_err_rows(hp.db[l].cpu().numpy()[None, :], db[None, :])
                    worst_w = max(worst_w, e, e_b)
                    assert e <= tol_bw and e_b <= tol_bw, f"dW[{l}] / db[{l}] iteration {it}: rel err {e:.3e} / {e_b:.3e}"
                dev_norms = {l: hp.gnorm[l][:nl[l]].cpu().numpy() for l in range(1, L)}
                for l in range(1, L):
                    np.testing.assert_allclose(dev_norms[l], O.row_norms(dHd[l]).astype(np.float32), rtol=5e-7, atol=1e-37)
                    # (b) end to end against the pure-oracle backward pass: a plausibility check, not the gate (the gate is (a),
                    #     every call on the same inputs at the plain bar): a ReLU output that is +0 on one side and a rounding
                    #     error above it on the other switches a whole gradient row on or off, so a few rows may differ
                    #     by more than any rounding bound; all the others must be within the depth-scaled bound
                    ref = bw["dH"][l]
                    den = np.maximum(np.abs(ref), np.abs(ref).max(axis=1, keepdims=True) / 16.0) + 1e-300
                    # (bf16: the forward rows differ by bf16 roundings between the sides, and so does which ReLU outputs are zero)
                    bad = (np.abs(dHd[l] - ref) / den).max(axis=1) > (REL_TOL_F32 if cd == "f32" else 4e-2) * 2 * (L - l + 1)
                    assert bad.mean() <= (0.01 if cd == "f32" else 0.05), f"dH[{l}] iteration {it} (end to end): {int(bad.sum())} of {len(bad)} rows off"
                    # the update itself, from the device's norms on both sides
                    rec["stats"][l] = O.cache_update(caches[l], it, mb.ids[l], rec["live"][l], rec["look"][l]["hit"], dev_norms[l],
                                                     p if it >= stabilization else 0.0, rec["H"][l])
            fused_now = fused and not hp.reads_rows_once(bt)      # whether this mini-batch's layer 0 was not looked up
            for l in range(L, 0 if fused_now else -1, -1):
                s, lk = snap["layers"][l], rec["look"][l]
                assert tuple(snap["counts"][l]) == lk["counts"], f"counts, iteration {it} layer {l}"
                assert np.array_equal(s["live"], rec["live"][l] if rec["live"][l] is not None else np.ones(len(mb.ids[l]), bool))
                assert np.array_equal(s["hit"], lk["hit"])
                assert np.array_equal(s["hit_pos"], lk["hit_pos"]) and np.array_equal(s["hit_slot"], lk["hit_slot"])
                assert np.array_equal(s["normal_pos"], lk["normal_pos"])
                if l >= 1:
                    assert np.array_equal(s["end"], mb.end[l]), f"pruned row ends, iteration {it} layer {l}"
                total_hits += len(lk["hit_pos"])
            # fused input: only the layer-1 nodes' own rows exist in H[0]
            ipos = rec["look"][1]["normal_pos"] if fused_now else rec["look"][0]["normal_pos"]
            if not fused_now:
                assert np.array_equal(snap["input_ids"], mb.ids[0][ipos])
            # gathered raw features: bit-exact
            rows_chk = ipos if sample_rows is None or len(ipos) <= sample_rows else np.sort(
                np.random.default_rng(it).choice(ipos, sample_rows, replace=False))
            # (GCN: the own rows enter the mean directly and are never stored; nor are they where layer 1's dense update
            #  reads them from the table itself)
            if not (fused_now and model == "gcn") and not hp.own_rows_from_table(bt):
                got0 = hp.H[0][torch.as_tensor(rows_chk.astype(np.int64), device="cuda")].cpu().numpy()
                want0 = rec["H"][0][rows_chk]
                differ = np.flatnonzero((got0.view(np.uint8) != want0.view(np.uint8)).any(axis=1))
                where = np.flatnonzero(got0[differ[0]] != want0[differ[0]]) if len(differ) else []
                assert len(differ) == 0, (f"gathered features, iteration {it}: {len(differ)} of {len(rows_chk)} rows differ, first at positions "
                                          f"{rows_chk[differ[:8]].tolist()}; in the first, columns {where[:8].tolist()} of {len(where)}: "
                                          f"{got0[differ[0]][where[:8]].tolist()} for {want0[differ[0]][where[:8]].tolist()}")
            # numerics: every computed row on every `check_numeric_every`-th iteration (and the last), a sample of the
            # computed rows of every layer on all the others
            full = it % check_numeric_every == 0 or it == iterations - 1
            tol = REL_TOL_F32 if w.compute_dtype == "f32" else 2e-2
            for l in range(1, L + 1):
                npos = rec["look"][l]["normal_pos"]
                if not full and len(npos) > 2048:
                    npos = np.sort(np.random.default_rng(77 * it + l).choice(npos, 2048, replace=False))
                out_dtype = "f32" if l == L else w.compute_dtype
                if len(npos):
                    idx = torch.as_tensor(npos.astype(np.int64), device="cuda")
                    got = G.to_f32(hp.H[l][idx])
                    # (a) each call against the oracle on the SAME inputs: the layer recomputed by the oracle from
                    #     the device's own previous-layer rows (bf16/fp16 values are exact in fp32)
                    # (fused input: the neighbours' rows were never materialised on the device; the oracle's
                    #  bit-identical feature rows take their place)
                    h_prev = rec["H"][0].astype(np.float32) if (fused and l == 1) else G.to_f32(hp.H[l - 1][:len(mb.ids[l - 1])])
                    agg64 = (O.aggregate_gcn if model == "gcn" else O.aggregate)(mb.start[l], mb.end[l], mb.col[l], npos, h_prev)
                    agg_dtype = "f32" if w.compute_dtype == "f32" else "bf16"
                    agg_want = O.round_to(agg64, agg_dtype).astype(np.float32)
                    agg_got = G.to_f32(hp.AGG[: len(npos) * dims[l - 1]].view(len(npos), dims[l - 1])) \
                        if (full and l == L and not hp.one_launch(l, bt.n[l])) else None
                    if full and model == "gcn" and l == L:   # the mean's halves: by position and in list order
                        hw = dims[l - 1] // 2
                        agg_got = np.concatenate([G.to_f32(hp.MEANPOS[: bt.n[l] * hw].view(bt.n[l], hw)[idx]),
                                                  G.to_f32(hp.AGG[: len(npos) * hw].view(len(npos), hw))], axis=1)
                    if agg_got is not None:        # the AGG buffer still holds the last layer's means
                        e_agg = T.rel_err_rows(agg_got, agg_want)
                        assert e_agg <= tol, f"AGG[{l}] iteration {it}: rel err {e_agg:.3e}"
                    h_self = h_prev[npos] if w.compute_dtype == "f32" else O.round_bf16(h_prev[npos])
                    if model == "gcn":
                        want_same = O.round_to(O.linear_gcn(agg_want, weights[l][0], weights[l][1], relu=(l < L)), out_dtype)
                    else:
                        want_same = O.round_to(O.linear(h_self, agg_want, weights[l][0], weights[l][1], relu=(l < L)), out_dtype)
                    e_same = T.rel_err_rows(got, want_same.astype(np.float32))
                    worst = max(worst, e_same)
                    tol_l = tol
                    if conditioned and model == "sage":
                        xw = np.abs(np.concatenate([h_self, agg_want], axis=1)).astype(np.float64) @ np.abs(weights[l][0]).astype(np.float64) \
                            + np.abs(weights[l][1])
                        ref64 = np.abs(want_same.astype(np.float64))
                        den = np.maximum(ref64, ref64.max(axis=1, keepdims=True) / 16.0)
                        den[den == 0] = 1.0
                        tol_l = max(tol, 4 * float((2.0 ** -24 * xw / den).max()))
                    assert e_same <= tol_l, f"H[{l}] iteration {it} (same inputs): rel err {e_same:.3e} (bound {tol_l:.2e})"
                    # (b) end to end against the pure-oracle pipeline: rounding differences of the layers below
                    #     propagate, so the bound grows with depth
                    e_e2e = T.rel_err_rows(got, rec["H"][l][npos].astype(np.float32))
                    worst_e2e = max(worst_e2e, e_e2e)
                    # (ill-conditioned narrow layers amplify what they inherit: there the same-inputs check is the gate)
                    assert conditioned or e_e2e <= tol * l, f"H[{l}] iteration {it} (end to end): rel err {e_e2e:.3e}"
                hpos = rec["look"][l]["hit_pos"]
                if len(hpos) and full:
                    # fetched rows are bit copies of the device cache, and match the oracle's cached rows within tolerance
                    got = G.to_f32(hp.H[l][torch.as_tensor(hpos.astype(np.int64), device="cuda")])
                    assert np.array_equal(got, pre_rows[l])
                    assert conditioned or T.rel_err_rows(got, rec["H"][l][hpos].astype(np.float32)) <= tol * l
            for l in range(1, L):
                if admit_budget and it >= stabilization:      # the estimates the update ranked by
                    assert np.array_equal(hp.saving[l][:len(mb.ids[l])].cpu().numpy(), rec["saving"][l]), f"estimates, iteration {it} layer {l}"
                st = rec["stats"][l]
                assert snap["stats"][l].tolist() == [st["admitted"], st["evicted_by_gradient"], st["overwritten"],
                                                     st["dropped_overflow"]], f"update stats, iteration {it} layer {l}"
        for l in range(1, L):
            exp = hp.export_cache(l, iterations)
            oc = caches[l]
            assert exp["head"] == oc.head
            # compare the valid set through the oracle's predicate, node by node
            for v, s, a in zip(exp["nodes"].tolist(), exp["slots"].tolist(), exp["stamps"].tolist()):
                assert oc.slot_of(v, iterations) == s and int(oc.slot_stamp[s]) == a
            filled = np.flatnonzero(oc.slot_node >= 0)
            n_valid = sum(1 for s in filled if oc.slot_of(int(oc.slot_node[s]), iterations) == s)
            assert n_valid == len(exp["nodes"])
        if bc is not None:
            # every feature row still intact on the oracle's side holds the same bytes in the device's buffer
            addr, nbytes = FGB.fg_cache_buffer(hp.cache)
            assert nbytes == bc.buffer_bytes
            wb = bc.feat_row_bytes
            intact = np.asarray([r for r, v in enumerate(hot) if bc.feature_rank(int(v)) == r], dtype=np.int64)
            if sample_rows is not None and len(intact) > sample_rows:
                intact = np.sort(np.random.default_rng(5).choice(intact, sample_rows, replace=False))
            from paper_2301_07482_amd.pipeline import _tensor_from_ptr
            lo = nbytes - len(hot) * wb
            region = _tensor_from_ptr(addr + lo, (len(hot), wb), torch.uint8, len(hot) * wb, "cuda")
            got = region[torch.as_tensor(len(hot) - 1 - intact, device="cuda")].cpu().numpy()
            want = np.stack([bc.buf[nbytes - (r + 1) * wb: nbytes - r * wb] for r in intact]) if len(intact) else got
            assert np.array_equal(got, want), "feature rows in the shared buffer"
            lost = len(hot) - sum(1 for r, v in enumerate(hot) if bc.feature_rank(int(v)) == r) if sample_rows is None else -1
            print(f"{w.name}: feature side served {served} input rows, {lost} of {len(hot)} rows displaced")
    finally:
        hp.close()
    print(f"{w.name}: worst rel err same-inputs {worst:.3e}, end-to-end {worst_e2e:.3e}" + (f", embedding gradients {worst_bw:.3e}, weight gradients {worst_w:.3e}" if backward else ""))
    if fs:
        return total_hits, worst, served
    return total_hits, worst


def test_iterations_tiny(env):
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    hits, worst = run_workload_parity(torch, w, w.iterations)
    print(f"tiny: {hits} hits over {w.iterations} iterations, worst rel err {worst:.3e}")
    assert hits > 100
    # the update as one call after the layers instead of its selection on a second stream beside them
    assert run_workload_parity(torch, w, w.iterations, overlap_update=False)[0] == hits
    # every mini-batch handed to the iteration before it: its top-down pass runs on the second stream beside that
    # iteration's layers, into the other set of lists
    assert run_workload_parity(torch, w, w.iterations, lookahead=True)[0] == hits
    assert run_workload_parity(torch, w, w.iterations, lookahead=True, fused=True, col_ids=True, admit_budget={1: 60})[0] > 0


def test_lookahead_promise_not_kept(env):
    """A mini-batch announced as the next one (its top-down pass is then already on the second stream) but not run next:
    the call that follows, for another mini-batch, still gives the sequential results."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = wl.WORKLOADS["tiny"]
    g = wl.make_graph(w)
    L = w.num_layers
    hp, weights, _ = G.make_hotpath(w, fused_input=True)
    ref, _, _ = G.make_hotpath(w, fused_input=True, overlap_update=False)
    try:
        def batch(it):
            mb = wl.minibatch(w, g, it)
            return DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)}, col_ids=True)
        for it in range(8):
            decoy = batch(100 + it) if it % 2 else None          # announced, never run
            hp.run(batch(it), it, next_bt=decoy)
            ref.run(batch(it), it)
            torch.cuda.synchronize()
            n = len(wl.minibatch(w, g, it).ids[L])
            assert torch.equal(hp.H[L][:n], ref.H[L][:n]), f"outputs, iteration {it}"
            for l in range(1, L):
                ea, eb = hp.export_cache(l, it + 1), ref.export_cache(l, it + 1)
                assert ea["head"] == eb["head"] and np.array_equal(ea["nodes"], eb["nodes"]) and np.array_equal(ea["slots"], eb["slots"])
    finally:
        hp.close()
        ref.close()


def test_iterations_queued_back_to_back_match_one_at_a_time(env):
    """Fourteen iterations of the medium workload queued without a synchronisation in between, each mini-batch announced
    to the iteration before it (so the second stream runs up to a step ahead, over three sets of lists and two halves of
    the update's workspace; in two of the iterations it is held back until layer 1 is done), leave the same outputs,
    counters, statistics and caches as the same iterations run one at a time on one stream."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = wl.WORKLOADS["medium"]
    g = wl.make_graph(w)
    L, K = w.num_layers, 14
    hp, weights, _ = G.make_hotpath(w, fused_input=True, fuse_small_layers=True, log_ring=K + 2)
    ref, _, _ = G.make_hotpath(w, fused_input=True, fuse_small_layers=True, overlap_update=False, log_ring=K + 2)
    try:
        assert hp.holds_second_stream() and not ref.holds_second_stream()
        mbs = [wl.minibatch(w, g, it) for it in range(K)]
        batches = [DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)}, col_ids=True) for it, mb in enumerate(mbs)]
        n_out = [len(mb.ids[L]) for mb in mbs]
        torch.cuda.synchronize()
        outs = []
        for it in range(K):
            hp.run(batches[it], it, next_bt=batches[it + 1] if it + 1 < K else None, hold_second_stream=it in (4, 9))
            outs.append(hp.H[L][:n_out[it]].clone())      # a copy on the same stream, in order: no synchronisation
        hp.flush()
        torch.cuda.synchronize()
        hits = 0
        for it in range(K):
            ref.run(batches[it], it)
            torch.cuda.synchronize()
            assert torch.equal(outs[it], ref.H[L][:n_out[it]]), f"outputs, iteration {it}"
            assert torch.equal(hp.counts_log[it], ref.counts_log[it]), f"counters, iteration {it}"
            assert torch.equal(hp.stats_log[it], ref.stats_log[it]), f"update statistics, iteration {it}"
            hits += int(ref.counts_log[it][1:L, 1].sum().item())
        assert hits > 1000, f"only {hits} cache hits: the caches were hardly used"
        for l in range(1, L):
            ea, eb = hp.export_cache(l, K), ref.export_cache(l, K)
            assert ea["head"] == eb["head"] and np.array_equal(ea["nodes"], eb["nodes"]) and np.array_equal(ea["slots"], eb["slots"]) \
                and np.array_equal(ea["stamps"], eb["stamps"])
            assert np.array_equal(hp.cache_rows(l, ea["slots"][:4000]), ref.cache_rows(l, eb["slots"][:4000])), f"cached rows, layer {l}"
    finally:
        hp.close()
        ref.close()


@pytest.mark.parametrize("order", ["roorooror", "oroorrooo", "rtoruotro"])
def test_steps_of_both_kinds_queued_back_to_back_match_one_at_a_time(env, order):
    """Steps whose selection goes with the loader (r), steps that put it on the second stream (o) and timed ones of both sizes, a call per layer
    (t, u), each announced to the one before it and queued without a synchronisation in between: the bits of the same steps run one at a time."""
    torch, B = env
    import dataclasses
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = dataclasses.replace(wl.WORKLOADS["tiny"], num_nodes=90_000, num_edges=1_800_000, feat_dim=52, hidden=128, fanouts=(3, 2, 8), batch=4501, cache_capacity=20_000)
    g = wl.make_graph(w)
    L = w.num_layers
    mbs = [wl.minibatch(w if k in "rt" else dataclasses.replace(w, batch=900), g, it) for it, k in enumerate(order)]
    paths = [G.make_hotpath(w, fused_input=True, fuse_small_layers=True)[0] for _ in range(2)]
    try:
        batches = [DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)}, col_ids=True) for it, mb in enumerate(mbs)]
        ends = [[None if e is None else e.clone() for e in bt.end] for bt in batches]
        outs = []
        for hp, alone in zip(paths, (False, True)):
            for bt, before in zip(batches, ends):      # (pruning empties rows of a mini-batch in place)
                for e, b in zip(bt.end, before):
                    if b is not None:
                        e.copy_(b)
            torch.cuda.synchronize()
            out = []
            for it, (k, bt) in enumerate(zip(order, batches)):
                hp.run(bt, it, next_bt=batches[it + 1] if it + 1 < len(order) else None, timer=(lambda *a: None) if k in "tu" else None)
                assert hp.loads_and_multiplies(bt) == (k in "rt")
                assert (hp._row_copy_due is None) == (hp._td_for is None) == (it + 1 == len(order))
                out += [hp.H[l][:len(mbs[it].ids[l])].clone() for l in range(1, L + 1)]
                if alone:
                    torch.cuda.synchronize()
            out += [hp.counts_log, hp.stats_log]
            for l in range(1, L):
                e = hp.export_cache(l, len(order))
                out += [torch.as_tensor(np.asarray(e[k])) for k in ("head", "nodes", "slots", "stamps")] + [torch.from_numpy(hp.cache_rows(l, e["slots"]))]
            assert int(hp.counts_log[:, 1:L, 1].sum()) > 1000, "the caches were hardly used"
            outs.append(out)
        assert len(outs[0]) == len(outs[1])
        for i, (a, b) in enumerate(zip(*outs)):
            assert torch.equal(a, b), f"record {i} of {len(outs[0])}"
    finally:
        for hp in paths:
            hp.close()


@pytest.mark.parametrize("workload,kwargs", [
    ("tiny", dict(fused_input=True)),
    ("tiny", dict(fused_input=True, copy_own_rows=True, fetch_with_loader=False)),
    ("tiny", dict(use_cache=False, fuse_small_layers=True)),
    ("tiny", dict(fused_input=True, overlap_update=False, fuse_small_layers=True)),
    ("tiny", dict(fused_input=True, backward=True, weight_grads=True)),
    ("tiny", dict(backward=True, weight_grads=True, overlap_update=False)),
    ("tiny", dict(fused_input=True, backward=True, fuse_small_layers=True)),
    ("tiny", dict(fused_input=True, backward=True, weight_grads=True, model="gcn")),
    ("tiny", dict(model="gcn")),
    ("host", dict(fused_input=True)),
    ("mixed", dict(fused_input=True)),
    ("mixed", dict(fused_input=True, backward=True, weight_grads=True)),
    ("mixed, few admitted", dict(fused_input=True, backward=True, weight_grads=True)),
    ("wide", dict(fused_input=True, backward=True, weight_grads=True)),
    # the update inside the weight gradients' launches: two of its workgroups for layer 1, nothing / everything admitted, more of them than
    # compute units are left free (the weight gradients are split otherwise then), and more than may wait for each other (own launches)
    ("two chunks", dict(fused_input=True, backward=True, weight_grads=True, overlap_update=False)),
    ("two chunks", dict(fused_input=True, backward=True, weight_grads=True, p_grad=0.0)),
    ("two chunks", dict(fused_input=True, backward=True, weight_grads=True, p_grad=1.0)),
    ("many chunks", dict(fused_input=True, backward=True, weight_grads=True, overlap_update=False)),
    ("too many chunks", dict(fused_input=True, backward=True, weight_grads=True)),
    # a step's update inside the loader's launch and the seed layer's: two of its workgroups for layer 1, nothing / everything admitted; fifteen
    ("two chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True)),
    ("two chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True, p_grad=0.0)),
    ("two chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True, p_grad=1.0)),
    ("two chunks of a step", dict(fused_input=True, overlap_update=False)),
    ("two chunks of a step", dict(fused_input=True, fuse_small_layers=True)),
    ("two chunks of a mixed step", dict(fused_input=True, overlap_update=False)),
    ("one piece a row, two chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True)),      # (own launches)
    ("one piece a row, two chunks of a mixed step", dict(fused_input=True, overlap_update=False)),
    ("two pieces a row, two chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True)),
    ("many chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True)),
    ("88 columns, many chunks of a step", dict(fused_input=True, overlap_update=False, fuse_small_layers=True)),
    ("many chunks of a step", dict(fused_input=True, fuse_small_layers=True)),      # (these two: with node ids as columns: in the launch that multiplies too)
])
@pytest.mark.parametrize("col_ids", [True, False])
def test_iteration_as_one_call_is_the_iteration_of_single_calls(env, workload, kwargs, col_ids):
    """`run` through fg_path_run and through the calls one by one: the same launches, so the same bits everywhere (embeddings, counters,
    statistics, gradients, cached rows). Announced mini-batches, one of them a promise that is not kept, one iteration without update."""
    torch, B = env
    import dataclasses
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = wl.WORKLOADS["tiny"]
    if workload == "host":       # 512 x 10 x 5 edges of 128 values: every input row is read once
        w = dataclasses.replace(w, feat_location="host", feat_dim=256, batch=512)
    if workload == "wide":       # weight gradients that take longer than the update (3 * 10^9 products, 2 MB of rows)
        w = dataclasses.replace(w, num_nodes=40_000, num_edges=1_200_000, feat_dim=256, hidden=512, fanouts=(4, 22), batch=512, p_grad=0.1)
    if workload.endswith(" step"):
        w = dataclasses.replace(w, num_nodes=40_000, num_edges=800_000, feat_dim=52, hidden=64, fanouts=(3, 2, 8), batch=301,
                                cache_capacity=5_000)
    if workload.startswith("88 columns"):
        workload, w = workload[12:], dataclasses.replace(w, hidden=88)
    if workload == "many chunks of a step":
        w = dataclasses.replace(w, num_nodes=90_000, batch=4501)
    if workload.endswith("mixed step"):
        w = dataclasses.replace(w, feat_dtype="f16", feat_dim=72, compute_dtype="bf16")
    pieces = {"one": 1, "two": 2}.get(workload.split(" ")[0], 0) if " a row" in workload else 0
    if pieces:
        w = dataclasses.replace(w, feat_dim=pieces * (8 if w.feat_dtype == "f16" else 4))
        workload = workload.split(", ")[1]
    if workload == "two chunks":
        w = dataclasses.replace(w, num_nodes=40_000, num_edges=800_000, feat_dim=52, hidden=88, fanouts=(3, 2, 8), batch=301, cache_capacity=5_000)
    if workload.endswith("many chunks"):
        w = dataclasses.replace(w, num_nodes=700_000, num_edges=16_000_000, feat_dim=16, hidden=16, fanouts=(2, 15, 20) if workload == "many chunks" else (1, 20, 20),
                                batch=1024 if workload == "many chunks" else 2048, cache_capacity=60_000)
    if workload == "mixed, few admitted":
        workload, w = "mixed", dataclasses.replace(w, p_grad=0.02)
    if workload == "mixed":      # wide enough for the upper layers' weight gradients to go ahead (8 Mi values in layer 1)
        w = dataclasses.replace(w, num_nodes=40_000, num_edges=1_200_000, feat_dim=72, feat_dtype="f16", compute_dtype="bf16", hidden=1280,
                                fanouts=(4, 22), batch=512)
    g = wl.make_graph(w)
    L, K, backward = w.num_layers, 7, kwargs.get("backward", False)
    paths = [G.make_hotpath(w, **kwargs)[0] for _ in range(2)]
    paths[1].runs_in_one_call = lambda: False
    try:
        assert paths[0].runs_in_one_call()
        mbs = [wl.minibatch(w, g, it) for it in range(K + 1)]

        def batch(it):
            mb = mbs[it]
            if backward:
                return DeviceBatch(mb, None, labels=wl.node_labels(w, mb.ids[L]), col_ids=col_ids)
            return DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)}, col_ids=col_ids)
        state, sums = [], []
        for hp in paths:
            batches = [batch(it) for it in range(K + 1)]
            if workload == "host":
                assert hp.reads_rows_once(batches[0])
            if workload == "mixed":
                assert hp.weight_grads_ahead(batches[0]) == backward
            rec = []
            for it in range(K):
                hp.run(batches[it], it, update=it != 4, next_bt=batches[K if it == 2 else it + 1] if it + 1 < K else None)
                n = mbs[it].ids
                if workload[:10] == "two chunks":
                    assert 4096 < len(n[1]) < 8192
                if workload.endswith(" step"):      # layer 1 as one launch from 24576 positions on; its selection in either loader: up to 32 chunks of 4096
                    assert (len(n[1]) >= 24576) == (workload[:4] == "many") and sum(-(-len(n[l]) // 4096) for l in range(1, L)) <= 32
                    one = workload[:4] == "many" and col_ids and w.feat_dtype == "f32" and (hp.overlap_update or w.hidden > 64)
                    assert hp.loads_and_multiplies(batches[it]) == one
                if workload.endswith("many chunks"):
                    groups = sum(-(-len(n[l]) // 4096) for l in range(1, L))
                    assert 32 < groups <= 64 if workload == "many chunks" else groups > 64
                rec += [hp.H[l][:len(n[l])].clone() for l in range(1, L + 1)]
                if backward:
                    rec += [hp.dH[l][:len(n[l])].clone() for l in range(1, L + 1)] + [x[:len(n[l])].clone() for l, x in enumerate(hp.gnorm) if l]
                if hp.weight_grads:
                    if workload == "many chunks":
                        sums.append([x.clone() for x in hp.dW[1:] + hp.db[1:]])
                    else:
                        rec += [x.clone() for x in hp.dW[1:] + hp.db[1:]]
                rec += [hp.live[l][:len(n[l])].clone() for l in range(1, L)] + [hp.counts.clone(), hp.stats.clone()]
            torch.cuda.synchronize()
            rec += [hp.counts_log, hp.stats_log, hp.input_log]
            if kwargs.get("use_cache", True):
                for l in range(1, L):
                    e = hp.export_cache(l, K)
                    rec += [torch.as_tensor(np.asarray(e[k])) for k in ("head", "nodes", "slots", "stamps")]
                    rec.append(torch.from_numpy(hp.cache_rows(l, e["slots"])))
            state.append(rec)
        assert len(state[0]) == len(state[1])
        for i, (a, b) in enumerate(zip(*state)):
            assert torch.equal(a, b), f"record {i} of {len(state[0])}"
        for it in range(len(sums) // 2):      # sums of the same products in another order: some 2^-24 of the result for each of a dozen additions in fp32
            for a, b in zip(sums[it], sums[it + len(sums) // 2]):
                assert (a - b).norm() <= 1e-6 * b.norm() and b.norm() > 0
    finally:
        for hp in paths:
            hp.close()


@pytest.mark.parametrize("rides,kwargs", [(True, dict(overlap_update=False)), (True, dict()), (False, dict())])
def test_a_failed_step_can_be_run_again(env, rides, kwargs):
    """A step whose seed layer is refused when its selection is queued already, with the loader or on the second stream: with the weights put right, it and
    the steps behind it are those of a model whose cache is empty."""
    torch, B = env
    import dataclasses
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = dataclasses.replace(wl.WORKLOADS["tiny"], num_nodes=90_000, num_edges=1_800_000, feat_dim=52, hidden=96, fanouts=(3, 2, 8), batch=4501 if rides else 900,
                            cache_capacity=20_000)
    g = wl.make_graph(w)
    L = w.num_layers
    paths = [G.make_hotpath(w, fused_input=True, fuse_small_layers=True, **kwargs)[0] for _ in range(2)]
    hp, ref = paths
    try:
        mbs = [wl.minibatch(w, g, it) for it in range(6)]
        make = lambda it: DeviceBatch(mbs[it], {l: wl.grad_norms(w, it, l, mbs[it].ids[l]) for l in range(1, L)}, col_ids=True)
        torch.cuda.synchronize()
        ahead = make(1)
        hp.run(make(0), 0, next_bt=ahead)
        good, hp.W[L] = hp.W[L], None
        with pytest.raises(B.FgError):
            hp.run(ahead, 1, next_bt=make(2))
        hp.W[L] = good
        outs = []
        for p in paths:
            out = []
            for it in range(1, 6):
                p.run(make(it), it)
                out += [p.H[l][:len(mbs[it].ids[l])].clone() for l in range(1, L + 1)] + [p.counts.clone(), p.stats.clone()]
            for l in range(1, L):
                e = p.export_cache(l, 6)
                out += [torch.as_tensor(np.asarray(e[k])) for k in ("nodes", "slots", "stamps")] + [torch.from_numpy(p.cache_rows(l, e["slots"]))]
            outs.append(out)
        for i, (a, b) in enumerate(zip(*outs)):
            assert torch.equal(a, b), f"record {i} of {len(outs[0])}"
    finally:
        for p in paths:
            p.close()


@pytest.mark.parametrize("kwargs", [dict(fused_input=True), dict(fused_input=True, backward=True, weight_grads=True),
                                    dict(backward=True, weight_grads=True, model="gcn")])
def test_iteration_as_one_call_uses_the_tensors_that_are_there(env, kwargs):
    """A caller puts other tensors in the places of a model's (its outputs, gradients, lists and logs) between two iterations: the next
    one reads and writes those, through fg_path_run as through the single calls, and leaves the earlier ones alone."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = wl.WORKLOADS["tiny"]
    g = wl.make_graph(w)
    L, backward = w.num_layers, kwargs.get("backward", False)
    paths = [G.make_hotpath(w, **kwargs)[0] for _ in range(2)]
    paths[1].runs_in_one_call = lambda: False
    names = ["H", "AGG_l"] + (["dH", "gnorm", "dW", "db"] if backward else []) + (["MEANPOS_l"] if kwargs.get("model") == "gcn" else [])
    try:
        records = []
        for hp in paths:
            def batch(it):
                mb = wl.minibatch(w, g, it)
                return DeviceBatch(mb, None, labels=wl.node_labels(w, mb.ids[L])) if backward else \
                    DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)})
            batches = [batch(it) for it in range(6)]
            for it in range(3):
                hp.run(batches[it], it)
            hp.flush()
            torch.cuda.synchronize()
            holders = [(getattr(hp, n), l) for n in names for l in range(len(getattr(hp, n)))]
            holders += [(lists[k], l) for lists in hp._lists for k in ("live", "hit", "hit_pos", "hit_slot", "normal_pos") for l in range(L + 1)]
            holders += [(lists, k) for lists in hp._lists for k in ("input_ids", "self_ids")]
            holders += [(hp.__dict__, k) for k in ("counts_log", "stats_log", "input_log", "ws_td", "ws_upd")]
            earlier = [(h[k], h[k].clone()) for h, k in holders if h[k] is not None]      # (kept: what may be written must stay allocated)
            for h, k in holders:
                if h[k] is not None:
                    h[k] = h[k].clone()
            for it in range(3, 6):
                hp.run(batches[it], it, next_bt=batches[it + 1] if it + 1 < 6 else None)
            hp.flush()
            torch.cuda.synchronize()
            assert all(torch.equal(was, now) for now, was in earlier), "a tensor that is not the model's any more was written"
            records.append([h[k].clone() for h, k in holders if h[k] is not None][:-2] + [torch.from_numpy(hp.cache_rows(l, hp.export_cache(l, 6)["slots"]))
                                                                                         for l in range(1, L)])
        for i, (a, b) in enumerate(zip(*records)):
            assert torch.equal(a, b), f"record {i} of {len(records[0])}"
    finally:
        for hp in paths:
            hp.close()


def test_refused_iteration_leaves_the_due_rows_and_the_announced_pass(env):
    """A call that is refused between two iterations (an iteration number that no call takes) changes nothing: the rows the one before admitted
    are copied by whoever comes next, a read-back or an iteration, and the next iteration waits for the pass announced."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = wl.WORKLOADS["tiny"]
    g = wl.make_graph(w)
    L, K = w.num_layers, 6
    hp, ref = (G.make_hotpath(w, fused_input=True)[0] for _ in range(2))
    try:
        def batch(it):
            mb = wl.minibatch(w, g, it)
            return DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)})
        mine, theirs = [batch(it) for it in range(K)], [batch(it) for it in range(K)]
        for it in range(K):
            nxt = it + 1 if it + 1 < K else None
            hp.run(mine[it], it, next_bt=mine[nxt] if nxt else None)
            ref.run(theirs[it], it, next_bt=theirs[nxt] if nxt else None)
            if nxt:
                assert hp._row_copy_due is not None
                with pytest.raises(B.FgError):
                    hp.run(mine[it], -1)
                assert hp._row_copy_due is not None
            if it % 2:
                hp.flush()
            assert torch.equal(hp.H[L], ref.H[L]) and torch.equal(hp.counts_log[it], ref.counts_log[it])
        for l in range(1, L):
            slots = [x.export_cache(l, K)["slots"] for x in (hp, ref)]
            assert np.array_equal(*slots) and np.array_equal(hp.cache_rows(l, slots[0]), ref.cache_rows(l, slots[1]))
    finally:
        hp.close()
        ref.close()


def test_cache_switched_off_while_admitted_rows_are_due(env):
    """`use_cache` off for one iteration behind one whose admitted rows are not copied yet: they are, and that iteration computes every row."""
    torch, B = env
    from paper_2301_07482_amd.pipeline import DeviceBatch
    w = wl.WORKLOADS["tiny"]
    g = wl.make_graph(w)
    L = w.num_layers
    paths = [G.make_hotpath(w, fused_input=True)[0] for _ in range(2)]
    paths[1].runs_in_one_call = lambda: False
    try:
        def batch(it):
            mb = wl.minibatch(w, g, it)
            return DeviceBatch(mb, {l: wl.grad_norms(w, it, l, mb.ids[l]) for l in range(1, L)})
        state = []
        for hp in paths:
            rec = []
            for it in range(5):
                hp.use_cache = it != 3
                hp.run(batch(it), it, next_bt=batch(it + 1) if it == 2 else None)      # (announced, but another object comes)
                assert (hp._row_copy_due is not None) == (it == 2)
                rec += [hp.H[L].clone(), hp.counts.clone()]
            assert int(rec[7][1:L, 1].sum()) == 0
            state.append(rec + [torch.from_numpy(hp.cache_rows(l, hp.export_cache(l, 5)["slots"])) for l in range(1, L)])
        assert all(torch.equal(a, b) for a, b in zip(*state))
    finally:
        for hp in paths:
            hp.close()


def test_device_sampled_iterations_queued_back_to_back(env):
    """Mini-batches sampled on the device (and their norms made there) on the current stream right before the call that
    announces them, twelve iterations queued without a synchronisation: the second stream, which runs ahead of the current
    one, must still read each mini-batch only after it is complete (the `ready` event). Same outputs, counters and
    statistics as the same iterations one at a time on one stream."""
    torch, B = env
    import dataclasses
    from fg_inputs import device as fdev, rng
    from paper_2301_07482_amd.pipeline import DeviceSampler
    w = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                            train_nodes=20_000, cache_capacity=20_000, t_stale=6)
    indptr, indices = fdev.chunglu_csr(wl.make_graph(w))
    L, K = w.num_layers, 12

    def sample(ds, it):
        seeds = torch.from_numpy(wl.seed_nodes(w, it).astype(np.int32)).cuda()
        bt = ds.sample(seeds, int(rng.make_key(w.seed, 0x5A3, it)), finish=False, ready=False)
        st = torch.cuda.current_stream()
        for l in range(1, L):
            bt.gnorm[l] = torch.empty(ds.bound[l], dtype=torch.float32, device="cuda")
            fdev.grad_norms(bt.ids[l], bt._counts.data_ptr() + 16 * l, ds.bound[l], int(rng.make_key(w.seed, 0x6AD, it, l)),
                            bt.gnorm[l], st.cuda_stream)
        bt.ready = torch.cuda.Event()
        bt.ready.record(st)
        return bt

    hp, _, feat = G.make_hotpath(w, fused_input=True, fuse_small_layers=True, p_grad=0.7, log_ring=K + 2)
    ref, _, _ = G.make_hotpath(w, feat_table=feat, fused_input=True, fuse_small_layers=True, p_grad=0.7, overlap_update=False, log_ring=K + 2)
    try:
        assert hp.holds_second_stream()
        ds = DeviceSampler(indptr, indices, w.num_nodes, w.fanouts, w.batch)
        torch.cuda.synchronize()
        outs, nxt = [], sample(ds, 0)
        for it in range(K):
            cur = nxt
            nxt = sample(ds, it + 1) if it + 1 < K else None
            hp.run(cur, it, next_bt=nxt)
            outs.append(hp.H[L][:w.batch].clone())
        hp.flush()
        torch.cuda.synchronize()
        hits = 0
        for it in range(K):
            ref.run(sample(ds, it), it)
            torch.cuda.synchronize()
            assert torch.equal(outs[it], ref.H[L][:w.batch]), f"outputs, iteration {it}"
            assert torch.equal(hp.counts_log[it], ref.counts_log[it]), f"counters, iteration {it}"
            assert torch.equal(hp.stats_log[it], ref.stats_log[it]), f"update statistics, iteration {it}"
            hits += int(ref.counts_log[it][1:L, 1].sum().item())
        assert hits > 0
    finally:
        hp.close()
        ref.close()


def test_iterations_tiny_layer_by_layer_top_down(env):
    """The same iterations with one fg_lookup_prune and one fg_cache_update call per layer instead of fg_top_down and
    fg_cache_update_all."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, 8, one_launch_top_down=False)[0] > 0
    assert run_workload_parity(torch, w, 8, one_launch_top_down=False, fused=True)[0] > 0


def test_iterations_tiny_degenerate_settings(env):
    """t_stale = 0 and p_grad = 0: no hit ever (Section 4.1.3), on the device as in the oracle."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, 6, t_stale=0)[0] == 0
    assert run_workload_parity(torch, w, 6, p_grad=0.0)[0] == 0


def test_iterations_tiny_stabilization_period(env):
    """Section 4.1.4: the first iterations run without the cache (no hit, nothing admitted), then it starts empty."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, 5, stabilization=5)[0] == 0
    assert run_workload_parity(torch, w, 14, stabilization=5)[0] > 0
    assert run_workload_parity(torch, w, 12, stabilization=4, one_launch_top_down=False, fused=True)[0] > 0


def test_iterations_gcn_layers(env):
    """GCN layers (propagation including the node itself, one weight matrix) through the same cached pipeline."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, 12, model="gcn")[0] > 50
    assert run_workload_parity(torch, w, 8, model="gcn", fused=True)[0] > 0
    import dataclasses
    w3 = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                             train_nodes=20_000, cache_capacity=20_000, t_stale=6)
    assert run_workload_parity(torch, w3, 8, p_grad=0.7, model="gcn", fused=True)[0] > 0


@pytest.mark.parametrize("dim,n,n_src,max_deg,seed", [(128, 700, 3000, 9, 0), (64, 50, 50, 4, 1), (8, 5, 9, 0, 2), (256, 300, 900, 40, 3)])
def test_aggregate_gcn_matches_oracle(env, dim, n, n_src, max_deg, seed):
    torch, B = env
    r = np.random.default_rng(seed)
    deg = r.integers(0, max_deg + 1, size=n)
    start = np.concatenate([[0], np.cumsum(deg)[:-1]]).astype(np.int32)
    end = (start + deg).astype(np.int32)
    col = np.concatenate([r.choice(n_src, size=k, replace=False) for k in deg] + [np.zeros(0, np.int64)]).astype(np.int32)
    rows = np.sort(r.permutation(n)[: max(1, n * 3 // 4)]).astype(np.int32)
    h = r.standard_normal((n_src, dim)).astype(np.float32)
    want = O.round_to(O.aggregate_gcn(start, end, col, rows, h), "f32")
    half = dim // 2
    pos = torch.full((n, half), 9.0, dtype=torch.float32, device="cuda")
    cmp_ = torch.full((n, half), 9.0, dtype=torch.float32, device="cuda")
    rows_dev = torch.zeros(n, dtype=torch.int32, device="cuda")
    rows_dev[:len(rows)] = dev(torch, rows)
    cnt = dev(torch, np.asarray([len(rows)], dtype=np.int64))
    tcol = dev(torch, col) if len(col) else torch.zeros(1, dtype=torch.int32, device="cuda")
    B.fg_aggregate_gcn(dev(torch, start), dev(torch, end), tcol, len(col), n, rows_dev, cnt, n, dev(torch, h), n_src, dim * 4, dim, pos, cmp_)
    got = np.concatenate([pos.cpu().numpy()[rows], cmp_.cpu().numpy()[:len(rows)]], axis=1)
    assert T.rel_err_rows(got, want) <= REL_TOL_F32
    untouched = np.setdiff1d(np.arange(n), rows)
    assert np.all(pos.cpu().numpy()[untouched] == 9.0) and np.all(cmp_.cpu().numpy()[len(rows):] == 9.0)
    # the same through the table-indexed variant: ids = a permutation of the table's rows
    perm = r.permutation(n_src).astype(np.int32)
    table = np.empty_like(h)
    table[perm] = h                                  # table[ids[j]] = h[j]
    pos.fill_(9.0)
    cmp_.fill_(9.0)
    B.fg_gather_aggregate_gcn(dev(torch, start), dev(torch, end), tcol, len(col), n, rows_dev, cnt, n, dev(torch, perm), n_src,
                              dev(torch, table), n_src, dim * 4, dim, pos, cmp_)
    got = np.concatenate([pos.cpu().numpy()[rows], cmp_.cpu().numpy()[:len(rows)]], axis=1)
    assert T.rel_err_rows(got, want) <= REL_TOL_F32


def test_iterations_one_launch_seed_layer(env):
    """The seed layer through fg_aggregate_linear (aggregation and dense update in one launch)."""
    torch, B = env
    import dataclasses
    from paper_2301_07482_amd import pipeline as P
    real = P.HotPath.__init__

    def patched(self, *a, **k):
        k["fuse_small_layers"] = True
        real(self, *a, **k)
    P.HotPath.__init__ = patched
    try:
        assert run_workload_parity(torch, wl.WORKLOADS["tiny"], 8)[0] > 0
        w3 = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                                 train_nodes=20_000, cache_capacity=20_000, t_stale=6)
        assert run_workload_parity(torch, w3, 6, p_grad=0.7, fused=True)[0] > 0
    finally:
        P.HotPath.__init__ = real


@pytest.mark.parametrize("seed", random_seeds(10))
def test_iterations_random_configurations(env, seed):
    """Depths 1 to 4, random widths (multiples of 4, so the tiled and the panel GEMMs both occur), fan-outs, batch sizes,
    cache sizes (down to rings that overflow), admission fractions and staleness bounds, in a random pipeline mode."""
    torch, B = env
    import dataclasses
    r = np.random.default_rng(1000 + seed)
    L = int(r.integers(1, 5))
    feat_dim = int(r.choice([8, 24, 32, 64, 100, 128]))
    # narrow layers are ill-conditioned for the 1e-5 metric (with 8 outputs after ReLU a row's largest value can be 1e-4 of
    # the terms it is summed from): the tolerance below takes the conditioning into account
    hidden = int(r.choice([8, 32, 40, 64, 96, 256]))
    w = dataclasses.replace(wl.WORKLOADS["tiny"], name=f"random/{seed}", num_nodes=int(r.integers(3_000, 40_000)),
                            num_edges=int(r.integers(20_000, 400_000)), feat_dim=feat_dim, hidden=hidden,
                            fanouts=tuple(int(x) for x in r.integers(1, 7, size=L)), batch=int(r.integers(1, 200)),
                            cache_capacity=int(r.choice([7, 60, 500, 5000])), t_stale=int(r.integers(0, 6)),
                            p_grad=float(r.choice([0.0, 0.2, 0.5, 0.9, 1.0])), seed=int(r.integers(1, 1 << 30)))
    fused = bool(r.integers(0, 2)) and feat_dim % 4 == 0
    one_launch = bool(r.integers(0, 2))
    print(f"L={L} dims {feat_dim}->{hidden} fanouts {w.fanouts} batch {w.batch} N={w.num_nodes} cap={w.cache_capacity} "
          f"t_stale={w.t_stale} p_grad={w.p_grad} fused={fused} one_launch_top_down={one_launch}", flush=True)
    run_workload_parity(torch, w, 9, fused=fused, one_launch_top_down=one_launch, conditioned=True)


@pytest.mark.parametrize("seed", random_seeds(10))
def test_iterations_random_configurations_widened(env, seed):
    """The options added around the core path, drawn at random together: mini-batches sampled on the device, block columns
    as node ids with the cache fetch inside or outside the loader's launch, access-aware admission with random budgets, a
    stabilization period; depths 2 to 4, random widths, fan-outs up to 12, rings that overflow."""
    torch, B = env
    import dataclasses
    r = np.random.default_rng(5000 + seed)
    L = int(r.integers(2, 5))
    feat_dim = int(r.choice([8, 32, 64, 128]))
    hidden = int(r.choice([32, 64, 96, 256]))
    w = dataclasses.replace(wl.WORKLOADS["tiny"], name=f"random-w/{seed}", num_nodes=int(r.integers(3_000, 40_000)),
                            num_edges=int(r.integers(20_000, 600_000)), feat_dim=feat_dim, hidden=hidden,
                            fanouts=tuple(int(x) for x in r.integers(1, 13, size=L)), batch=int(r.integers(1, 120)),
                            cache_capacity=int(r.choice([7, 60, 500, 5000])), t_stale=int(r.integers(1, 6)),
                            p_grad=float(r.choice([0.2, 0.5, 0.9, 1.0])), seed=int(r.integers(1, 1 << 30)))
    kw = dict(fused=bool(r.integers(0, 2)), device_sampler=bool(r.integers(0, 2)), fetch_with_loader=bool(r.integers(0, 2)),
              stabilization=int(r.choice([0, 0, 3])), overlap_update=bool(seed % 2), lookahead=bool((seed // 2) % 2))
    kw["col_ids"] = kw["fused"] and bool(r.integers(0, 2))
    if r.integers(0, 2):
        kw["admit_budget"] = {l: int(r.choice([1, 5, 40, 400])) for l in range(1, L)}
    print(f"L={L} dims {feat_dim}->{hidden} fanouts {w.fanouts} batch {w.batch} N={w.num_nodes} E={w.num_edges} cap={w.cache_capacity} "
          f"t_stale={w.t_stale} p_grad={w.p_grad} {kw}", flush=True)
    run_workload_parity(torch, w, 9, conditioned=True, **kw)


@pytest.mark.parametrize("seed", random_seeds(6))
def test_iterations_random_feature_side(env, seed):
    """Random depths, row widths, ring sizes, buffer sizes and hot-list lengths for the bidirectional cache, with the
    table rows of the cached nodes negated after the fill: ranks, gathered rows and buffer contents are compared bit for bit."""
    torch, B = env
    import dataclasses
    r = np.random.default_rng(2000 + seed)
    L = int(r.integers(2, 5))
    feat_dim = int(r.choice([8, 24, 64, 100, 128]))
    hidden = int(r.choice([32, 64, 96]))
    cap = int(r.choice([40, 300, 2000]))
    w = dataclasses.replace(wl.WORKLOADS["tiny"], name=f"random-fs/{seed}", num_nodes=int(r.integers(3_000, 30_000)),
                            num_edges=int(r.integers(20_000, 300_000)), feat_dim=feat_dim, hidden=hidden,
                            fanouts=tuple(int(x) for x in r.integers(1, 6, size=L)), batch=int(r.integers(8, 150)),
                            cache_capacity=cap, t_stale=int(r.integers(1, 6)), p_grad=float(r.choice([0.3, 0.7, 1.0])),
                            seed=int(r.integers(1, 1 << 30)))
    rings = G.rings_bytes(w)
    buffer_bytes = -(-int(rings * r.uniform(1.0, 1.6)) // 256) * 256 + 256 * int(r.integers(0, 8))
    n_hot = int(min(w.num_nodes, (buffer_bytes // (feat_dim * 4)) * r.uniform(0.3, 1.0)))
    fused = bool(r.integers(0, 2))
    print(f"L={L} dims {feat_dim}->{hidden} cap={cap} rings={rings} buffer={buffer_bytes} n_hot={n_hot} fused={fused}", flush=True)
    hits, worst, served = run_workload_parity(torch, w, 8, fused=fused, conditioned=True,
                                              feature_side=dict(n_hot=n_hot, buffer_bytes=buffer_bytes, poison=True))
    assert served > 0


def test_iterations_tiny_small_ring(env):
    """A cache much smaller than a layer: wrap-around and overflow every iteration."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    hits, _ = run_workload_parity(torch, w, 10, capacity=97, p_grad=0.9)
    assert hits > 0


rings_end = G.rings_bytes


@pytest.mark.parametrize("fused", [False, True])
def test_iterations_tiny_feature_side_displaced_by_the_ring(env, fused):
    """Bidirectional cache (Section 4.2): the buffer starts full of raw features (every byte of it, the ring's included)
    and the ring eats into them as it fills. The table rows of the cached nodes are negated after the fill, so every
    row the loader takes from the wrong place fails the bit comparison of H[0] or the numerics."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    cap = 1500                                        # rows of 256 bytes on both sides: the ring overlays ranks 524 .. 2023
    buffer_bytes = cap * 256 + 524 * 256 + 256
    n_hot = buffer_bytes // 256
    hits, worst, served = run_workload_parity(torch, w, 14, capacity=cap, p_grad=0.3, fused=fused,
                                              feature_side=dict(n_hot=n_hot, buffer_bytes=buffer_bytes, poison=True))
    assert hits > 0 and served > 500


def test_iterations_three_layers_feature_side_two_rings_unaligned_rows(env):
    """Two rings of 1 KB rows against feature rows of 400 bytes (the medium workload's widths on a small graph): feature
    rows straddle slot ends and the start of the second ring."""
    torch, B = env
    import dataclasses
    w = dataclasses.replace(wl.WORKLOADS["medium"], name="medium/small", num_nodes=60_000, num_edges=1_500_000, batch=64,
                            cache_capacity=700, t_stale=4)
    end = rings_end(w)
    buffer_bytes = -(-(end + 300 * 400) // 256) * 256
    n_hot = buffer_bytes // 400
    for fused in (False, True):
        hits, worst, served = run_workload_parity(torch, w, 9, p_grad=0.8, fused=fused,
                                                  feature_side=dict(n_hot=n_hot, buffer_bytes=buffer_bytes, poison=True))
        assert hits > 0 and served > 0


def test_feature_side_state_rules(env):
    """Features go into an empty cache only; a clear drops them; the row width must match."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    hot = wl.make_graph(w).hottest(64)
    hp, _, feat = G.make_hotpath(w, hot_ids=hot, buffer_bytes=rings_end(w) + 64 * 256)
    try:
        ids = dev(torch, hot[:10].astype(np.int32))
        assert hp.feature_ranks(ids, 10)[0].tolist() == list(range(10))
        out = torch.zeros((10, 32), dtype=torch.float32, device="cuda")
        with pytest.raises(B.FgError) as e:           # half-width rows
            B.fg_gather_features(hp.cache, feat, w.num_nodes, 256, 128, ids, None, None, 10, out, 10, 128)
        assert e.value.code == B.FG_ERR_SHAPE
        from paper_2301_07482_amd.pipeline import DeviceBatch
        mb = wl.minibatch(w, wl.make_graph(w), 0)
        hp.run(DeviceBatch(mb, {1: wl.grad_norms(w, 0, 1, mb.ids[1])}), 0)
        with pytest.raises(B.FgError) as e:           # the embedding side is no longer empty
            B.fg_cache_fill_features(hp.cache, ids, 10, feat, w.num_nodes, 256, 256)
        assert e.value.code == B.FG_ERR_STATE
        B.fg_cache_clear(hp.cache)
        assert B.fg_cache_feature_rows(hp.cache) == 0
        assert hp.feature_ranks(ids, 10)[0].tolist() == [-1] * 10
        B.fg_cache_fill_features(hp.cache, ids, 10, feat, w.num_nodes, 256, 256)
        assert hp.feature_ranks(ids, 10)[0].tolist() == list(range(10))
        bad = dev(torch, np.asarray([5, -1, w.num_nodes, 7], dtype=np.int32))     # ids out of range leave their rank unused
        B.fg_cache_fill_features(hp.cache, bad, 4, feat, w.num_nodes, 256, 256)
        probe = dev(torch, np.asarray([5, 7, -1, w.num_nodes, 6], dtype=np.int32))
        assert hp.feature_ranks(probe, 5)[0].tolist() == [0, 3, -1, -1, -1]
    finally:
        hp.close()


def test_iterations_tiny_fused_input(env):
    """Layer 1 aggregated straight from the feature table (fg_gather_aggregate): same lists, same outputs."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    hits, worst = run_workload_parity(torch, w, w.iterations, fused=True)
    assert hits > 100


def test_iterations_fused_input_with_node_ids_as_block_columns(env):
    """The fused loader given block 1 with node ids as columns (fg_gather_aggregate_ids), with the fetch of the cached
    embeddings inside its launch (one and two cached layers) and as a launch of its own."""
    torch, B = env
    for ride in (True, False):
        assert run_workload_parity(torch, wl.WORKLOADS["tiny"], 10, fused=True, col_ids=True, fetch_with_loader=ride)[0] > 0
        assert run_workload_parity(torch, wl.WORKLOADS["medium"], 4, check_numeric_every=2, sample_rows=20000, fused=True, col_ids=True,
                                   fetch_with_loader=ride)[0] > 0
    # the loader's copy of the layer-1 nodes' own rows (what the dense update reads where it cannot take them from the table)
    assert run_workload_parity(torch, wl.WORKLOADS["tiny"], 10, fused=True, col_ids=True, copy_own_rows=True)[0] > 0
    assert run_workload_parity(torch, wl.WORKLOADS["medium"], 4, check_numeric_every=2, sample_rows=20000, fused=True, col_ids=True,
                               copy_own_rows=True)[0] > 0


def test_iterations_access_aware_admission(env):
    """Whole iterations with the access-aware admission on both sides: estimates, admitted sets, cache state and outputs.
    Budgets small enough that rows are turned away in every update; two and three layers; with the fused loader."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, w.iterations, admit_budget={1: 40})[0] > 0
    assert run_workload_parity(torch, w, 12, fused=True, col_ids=True, admit_budget={1: 150}, t_stale=6, p_grad=0.9)[0] > 0
    w = wl.WORKLOADS["medium"]
    assert run_workload_parity(torch, w, 5, check_numeric_every=2, sample_rows=20000, fused=True, col_ids=True,
                               admit_budget={1: 3000, 2: 400}, p_grad=0.9)[0] > 0


def test_device_csr_is_the_host_graph_up_to_pow_rounding(env):
    """The CSR the device writes for a synthetic graph is the host's graph: same degrees and the same neighbour at every
    slot, except where the device's pow and numpy's differ in the last place right at a rounding boundary."""
    torch, B = env
    from fg_inputs import device as fdev
    w = wl.WORKLOADS["tiny"]
    g = wl.make_graph(w)
    indptr_t, indices_t = fdev.chunglu_csr(g)
    indptr, indices = indptr_t.cpu().numpy(), indices_t.cpu().numpy()
    nodes = np.arange(w.num_nodes)
    deg = g.degree(nodes)
    assert (np.diff(indptr) != deg).mean() < 1e-3 and abs(int(indptr[-1]) - w.num_edges) < 0.05 * w.num_edges
    same = np.flatnonzero(np.diff(indptr) == deg)
    v = np.repeat(same, deg[same])
    slot = np.arange(len(v)) - np.repeat(np.cumsum(deg[same]) - deg[same], deg[same])
    at = indptr[v] + slot
    assert (indices[at] != g.neighbour(v, slot)).mean() < 1e-3
    assert indices.min() >= 0 and indices.max() < w.num_nodes


def _local_csr(torch, indptr_t, indices_t, nodes):
    """The rows of `nodes` out of a CSR in device memory, as something the oracle's sampler can index: a dictionary
    v -> first entry, v + 1 -> one past the last, into a short array holding just those rows (in node order)."""
    order = np.unique(np.asarray(nodes, dtype=np.int64))
    t = torch.from_numpy(order).cuda()
    lo, hi = indptr_t[t], indptr_t[t + 1]
    length = hi - lo
    total = int(length.sum().item())
    first = torch.cumsum(length, 0) - length
    at = torch.repeat_interleave(lo, length) + (torch.arange(total, device="cuda") - torch.repeat_interleave(first, length))
    rows = indices_t[at].cpu().numpy() if total else np.zeros(0, dtype=np.int32)
    first, length = first.cpu().numpy(), length.cpu().numpy()
    indptr = {}
    for v, a, d in zip(order.tolist(), first.tolist(), length.tolist()):
        indptr[v] = a
        indptr[v + 1] = a + d
    return indptr, rows


def test_sampler_at_full_size(env):
    """fg_sample_block on the large workload's graph (111 M nodes, 1.6 G edges as a CSR in HBM), in the configuration
    bench.py --device-sampler runs: batch 1024, fan-outs 15/10/5. Every block of two mini-batches against the oracle's
    sampler, which is handed the rows of the layer's nodes copied out of the same CSR; bit for bit."""
    torch, B = env
    from fg_inputs import device as fdev, rng
    from oracle import sampler_oracle as S
    from paper_2301_07482_amd.pipeline import DeviceSampler
    w = wl.WORKLOADS["large_hbm"]
    indptr_t, indices_t = fdev.chunglu_csr(wl.make_graph(w))
    assert abs(int(indices_t.numel()) - w.num_edges) < 0.01 * w.num_edges
    sampler = DeviceSampler(indptr_t, indices_t, w.num_nodes, w.fanouts, w.batch)
    L = w.num_layers
    for it in (0, 7):
        seeds = wl.seed_nodes(w, it)
        key = int(rng.make_key(w.seed, 0x5A3, it))
        bt = sampler.sample(dev(torch, seeds.astype(np.int32)), key)
        cur = [int(v) for v in seeds]
        for l in range(L, 0, -1):
            indptr, rows = _local_csr(torch, indptr_t, indices_t, cur)
            start, end, col, col_ids, below = S.sample_block(indptr, rows, cur, int(w.fanouts[l - 1]), S.layer_key(key, l))
            assert bt.n[l - 1] == len(below) and bt.nnz[l] == len(col)
            assert bt.ids[l - 1].cpu().numpy()[:len(below)].tolist() == below, f"nodes of layer {l - 1}, mini-batch {it}"
            assert bt.start[l].cpu().numpy()[:len(cur)].tolist() == start and bt.end[l].cpu().numpy()[:len(cur)].tolist() == end
            assert bt.col[l].cpu().numpy()[:len(col)].tolist() == col, f"columns of block {l}, mini-batch {it}"
            if l == 1:
                assert bt.col_ids1.cpu().numpy()[:len(col)].tolist() == col_ids
            cur = below
        print(f"mini-batch {it}: layers {bt.n}, edges {bt.nnz[1:]}")
        assert bt.n[0] > 300_000 and bt.nnz[1] > 400_000


def test_device_gradient_norms_are_the_host_recipe(env):
    """The synthetic gradient norms made on the device from node ids (for loops that sample there) are those of
    workload.grad_norms up to the last place of the device's log / cos / exp; a device-side count cuts the list."""
    torch, B = env
    from fg_inputs import device as fdev, rng
    w = wl.WORKLOADS["tiny"]
    ids = np.random.default_rng(0).permutation(w.num_nodes)[:3000].astype(np.int32)
    want = wl.grad_norms(w, 5, 1, ids)
    out = torch.full((3000,), -1.0, device="cuda")
    cnt = torch.tensor([2500], dtype=torch.int64, device="cuda")
    fdev.grad_norms(dev(torch, ids), cnt.data_ptr(), 3000, int(rng.make_key(w.seed, 0x6AD, 5, 1)), out, None)
    got = out.cpu().numpy()
    np.testing.assert_allclose(got[:2500], want[:2500], rtol=2e-6)
    assert np.all(got[2500:] == -1.0)


def test_iterations_on_device_sampled_minibatches(env):
    """The mini-batches come from fg_sample_block (the graph written out as a CSR in HBM, the oracle sampling from a copy
    of it): sampled nodes and blocks bit for bit, then the whole iteration on them as in the other tests."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, w.iterations, fused=True, col_ids=True, device_sampler=True)[0] > 0
    assert run_workload_parity(torch, w, 6, device_sampler=True)[0] > 0
    # with the backward pass on transposed blocks built on the device; three layers
    assert run_workload_parity(torch, w, 6, fused=True, device_sampler=True, backward=True)[0] > 0
    import dataclasses
    w3 = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                             train_nodes=20_000, cache_capacity=20_000, t_stale=6)
    assert run_workload_parity(torch, w3, 8, p_grad=0.7, fused=True, device_sampler=True, backward=True)[0] > 0


def test_iterations_with_layer_sizes_left_on_the_device(env):
    """Device-sampled mini-batches run without their sizes ever reaching the host beforehand: every call gets the sampler's
    bounds and, where it walks a whole layer, the address of the layer's count. Same results as with host sizes."""
    torch, B = env
    w = wl.WORKLOADS["tiny"]
    assert run_workload_parity(torch, w, w.iterations, fused=True, device_sampler=True, device_counts=True)[0] > 0
    assert run_workload_parity(torch, w, 6, device_sampler=True, device_counts=True)[0] > 0      # input layer bounded by the node count
    assert run_workload_parity(torch, w, 6, fused=True, device_sampler=True, device_counts=True, lookahead=True)[0] > 0
    import dataclasses
    w3 = dataclasses.replace(wl.WORKLOADS["large_hbm"], name="large_hbm/small", num_nodes=200_000, num_edges=4_000_000, batch=128,
                             train_nodes=20_000, cache_capacity=20_000, t_stale=6)
    assert run_workload_parity(torch, w3, 8, p_grad=0.7, fused=True, device_sampler=True, device_counts=True, backward=True)[0] > 0
    assert run_workload_parity(torch, w3, 6, p_grad=0.7, fused=True, device_sampler=True, device_counts=True, model="gcn")[0] > 0
    assert run_workload_parity(torch, w3, 6, p_grad=0.7, fused=True, device_sampler=True, device_counts=True,
                               admit_budget={1: 300, 2: 40})[0] > 0


def test_iterations_medium_fused_input(env):
    torch, B = env
    w = wl.WORKLOADS["medium"]
    hits, worst = run_workload_parity(torch, w, 6, check_numeric_every=2, sample_rows=20000, fused=True)
    assert hits > 0


def test_iterations_medium(env):
    torch, B = env
    w = wl.WORKLOADS["medium"]
    hits, worst = run_workload_parity(torch, w, 8, check_numeric_every=4, sample_rows=20000)
    print(f"medium: {hits} hits, worst rel err {worst:.3e}")
    assert hits > 0


def test_iterations_large_hbm_full_size(env):
    """The benchmarked workload at its full size (111 M nodes, 57 GB table in HBM, 2 x 11.1 M cache slots) in the launch
    configuration bench.py times (fused loader, whole-pass top-down, seed layer in one launch, fetch and update calls), more iterations than the
    staleness bound so that entries age out; index work compared in full every iteration, numerics on a row sample every
    iteration and in full every 8th. (The layer-1 dense update reads the nodes' own rows from the table here; the loader's
    copy of them is compared bit for bit in the tests that ask for it with copy_own_rows, and at this size in the test
    with the backward pass, whose weight gradients need it.)"""
    torch, B = env
    w = wl.WORKLOADS["large_hbm"]
    hits, worst = run_workload_parity(torch, w, 24, check_numeric_every=8, sample_rows=20000, fused=True, col_ids=True, lookahead=True,
                                      fuse_small_layers=True)
    print(f"large_hbm: {hits} hits, worst rel err {worst:.3e}")
    assert hits > 1000


def test_iterations_large_hbm_full_size_separate_calls(env):
    """The same workload through the per-layer calls (fg_lookup_prune incl. layer 0, fg_gather of every surviving input
    row, fg_aggregate for layer 1, fg_gather of cached rows, fg_cache_update per layer)."""
    torch, B = env
    w = wl.WORKLOADS["large_hbm"]
    hits, worst = run_workload_parity(torch, w, 8, check_numeric_every=4, sample_rows=20000, one_launch_top_down=False)
    print(f"large_hbm, separate calls: {hits} hits, worst rel err {worst:.3e}")
    assert hits > 0


def test_iterations_large_host_resident(env):
    """Same graph with the feature table in pinned host memory, read zero-copy over the host link by the fused loader
    (the configuration bench.py --workload large_host times)."""
    torch, B = env
    w = wl.WORKLOADS["large_host"]
    hits, worst = run_workload_parity(torch, w, 6, check_numeric_every=5, sample_rows=20000, fused=True)
    print(f"large_host: {hits} hits, worst rel err {worst:.3e}")
    assert hits > 0


def test_iterations_large_host_resident_feature_side(env):
    """The host-resident workload with the raw features of the 300,000 hottest nodes on the feature side of the caches'
    buffer (the configuration bench.py --workload large_host --feature-rows times, with fewer rows so that the CPU side
    stays within minutes): ranks and gathered rows compared on samples, index work in full."""
    torch, B = env
    w = wl.WORKLOADS["large_host"]
    n_hot = 300_000
    buffer_bytes = -(-(rings_end(w) + n_hot * 512) // 256) * 256
    hits, worst, served = run_workload_parity(torch, w, 4, check_numeric_every=3, sample_rows=20000, fused=True,
                                              feature_side=dict(n_hot=n_hot, buffer_bytes=buffer_bytes))
    print(f"large_host with feature side: {hits} hits, {served} input rows from the buffer, worst rel err {worst:.3e}")
    assert served > 10000


def test_iterations_large_host_resident_separate_gather(env):
    """The host-resident table through fg_gather (every surviving input row copied to HBM first)."""
    torch, B = env
    w = wl.WORKLOADS["large_host"]
    hits, worst = run_workload_parity(torch, w, 3, check_numeric_every=2, sample_rows=20000)
    print(f"large_host, separate gather: {hits} hits, worst rel err {worst:.3e}")


@pytest.mark.parametrize("model,backward,device_sampler", [("sage", False, False), ("sage", False, True), ("sage", True, True), ("gcn", False, False)])
def test_iterations_host_table_rows_read_once(env, model, backward, device_sampler):
    """A host table under the fused loader, on both sides of the size from which every input row is read once into HBM (a
    mini-batch of four seeds stays with the fused loader): everything as the oracle has it. With the device's sampler the
    larger mini-batch's bound on its input layer exceeds the node count (announced ahead in the case without backward pass)."""
    torch, B = env
    import dataclasses
    from paper_2301_07482_amd.pipeline import HotPath
    base = wl.WORKLOADS["medium"]
    for batch, once in ((4, False), (256, True)):
        w = dataclasses.replace(base, num_nodes=60_000, num_edges=900_000, batch=batch, cache_capacity=9000, feat_location="host",
                                t_stale=3, feat_dim=104)
        seen = []
        plain = HotPath.reads_rows_once
        HotPath.reads_rows_once = lambda self, bt: seen.append(plain(self, bt)) or seen[-1]
        try:
            hits, worst = run_workload_parity(torch, w, 6, fused=True, col_ids=model == "sage" and not device_sampler, lookahead=not backward,
                                              model=model, backward=backward, device_sampler=device_sampler, device_counts=device_sampler)
        finally:
            HotPath.reads_rows_once = plain
        assert seen and all(s == once for s in seen), (batch, seen)
        print(f"host table, batch {batch}, {model}: {hits} hits, worst rel err {worst:.3e}")


# ------------------------------------------------------------------------------------------------ bf16 path

@pytest.mark.parametrize("src,d_in,d_out,n_rows,max_rows,relu,out", [("f16", 768, 1024, 700, 900, True, "bf16"),
                                                                     ("bf16", 1024, 1024, 300, 300, False, "f32"),
                                                                     ("bf16", 64, 72, 129, 200, True, "bf16"),
                                                                     ("f16", 8, 8, 5, 130, False, "f32"),
                                                                     ("bf16", 64, 1024, 3900, 4096, True, "bf16"),     # 64 x 128 tiles
                                                                     ("f16", 128, 512, 17000, 17000, False, "f32")])   # 128 x 128 tiles
def test_linear_bf16_matches_oracle(env, src, d_in, d_out, n_rows, max_rows, relu, out):
    torch, B = env
    r = np.random.default_rng(d_in + d_out)
    n_src = max_rows + 300
    code = {"f16": B.FG_F16, "bf16": B.FG_BF16, "f32": B.FG_F32}
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
    h = O.round_to(r.standard_normal((n_src, d_in)), src).astype(np.float32)
    agg = O.round_bf16(r.standard_normal((max_rows, d_in)) * 0.3)
    W = O.round_bf16(r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in))
    bias = (0.1 * r.standard_normal(d_out)).astype(np.float32)
    rows = np.sort(r.permutation(n_src)[:max_rows]).astype(np.int32)
    up = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).cuda().to(tdt[dt])
    t_out = torch.full((n_src, d_out), -3.0, dtype=tdt[out], device="cuda")
    t_cnt = torch.tensor([n_rows], dtype=torch.int64, device="cuda")
    osz = 2 if out == "bf16" else 4
    B.fg_linear(up(h, src), n_src, d_in * 2, code[src], up(agg, "bf16"), d_in * 2, dev(torch, rows), t_cnt, max_rows, d_in,
                d_out, up(W, "bf16"), B.FG_BF16, dev(torch, bias), 1 if relu else 0, t_out, n_src, d_out * osz, code[out], None)
    got = G.to_f32(t_out)
    sel = rows[:n_rows]
    want = O.round_to(O.linear(O.round_bf16(h[sel]), agg[:n_rows], W, bias, relu), out).astype(np.float32)
    untouched = np.ones(n_src, bool)
    untouched[sel] = False
    assert np.all(got[untouched] == -3.0)
    err = T.rel_err_rows(got[sel], want)
    print(f"linear bf16 {src} {d_in}x{d_out}: rel err {err:.3e}")
    assert err <= 2e-2
    # identity panels: exact, and wrong for any operand-layout mistake
    if d_in == d_out:
        I, Z = np.eye(d_in, dtype=np.float32), np.zeros((d_in, d_in), np.float32)
        for Wp, ref in [(np.vstack([I, Z]), O.round_bf16(h[sel])), (np.vstack([Z, I]), agg[:n_rows])]:
            t2 = torch.zeros((n_src, d_out), dtype=torch.float32, device="cuda")
            B.fg_linear(up(h, src), n_src, d_in * 2, code[src], up(agg, "bf16"), d_in * 2, dev(torch, rows), t_cnt, max_rows,
                        d_in, d_out, up(Wp, "bf16"), B.FG_BF16, None, 0, t2, n_src, d_out * 4, B.FG_F32, None)
            assert np.array_equal(t2.cpu().numpy()[sel], ref)


@pytest.mark.parametrize("d_in,d_out,n_rows", [(8, 8, 1), (56, 72, 63), (64, 64, 64), (72, 200, 65), (128, 136, 700), (264, 24, 130),
                                               (128, 64, 65), (136, 200, 65), (192, 72, 1), (120, 72, 100), (128, 256, 8192), (128, 256, 8193)])
@pytest.mark.parametrize("src", ["f16", "bf16"])
def test_linear_bf16_transposed_weights_small_tile(env, src, d_in, d_out, n_rows):
    """The 64 x 64 tile with weights as [N x K], whose wavefronts share each step of 128 k values (128 input columns and more, at
    most 512 workgroups) or not: contractions of a fraction of a step, of whole steps and with a remainder in either half; exact on
    identity panels."""
    torch, B = env
    r = np.random.default_rng(d_in + d_out + n_rows)
    n_src = n_rows + 9
    tdt, code = (torch.float16, B.FG_F16) if src == "f16" else (torch.bfloat16, B.FG_BF16)
    h = dev(torch, r.standard_normal((n_src, d_in)).astype(np.float32)).to(tdt)
    agg = dev(torch, r.standard_normal((n_rows, d_in)).astype(np.float32)).bfloat16()
    rows = dev(torch, np.sort(r.permutation(n_src)[:n_rows]).astype(np.int32))
    bias = dev(torch, r.standard_normal(d_out).astype(np.float32))
    x = torch.cat([h[rows.long()].bfloat16(), agg], 1).double()
    W = dev(torch, (r.standard_normal((2 * d_in, d_out)) / np.sqrt(2 * d_in)).astype(np.float32)).bfloat16()
    eye = torch.zeros((2 * d_in, d_out), device="cuda")
    k = torch.arange(d_out, device="cuda")
    eye[(k * 7) % (2 * d_in), k] = 1.0
    for weights, exact in ((W, False), (eye.bfloat16(), True)):
        out = torch.full((n_src, d_out), -3.0, device="cuda")
        B.fg_linear_wt(h, n_src, d_in * 2, code, agg, d_in * 2, rows, None, n_rows, d_in, d_out, weights.t().contiguous(), B.FG_BF16,
                       None if exact else bias, 0, out, n_src, d_out * 4, B.FG_F32)
        want = x @ weights.double() + (0.0 if exact else bias.double())
        got = out[rows.long()].double()
        # bf16 products are exact in fp32; a sum of at most 528 of them, 16 at a time, is off by a few half-ulps
        assert bool((got == want).all()) if exact else float((got - want).norm() / want.norm()) <= 8 * 2.0 ** -24
        out[rows.long()] = -3.0
        assert bool((out == -3.0).all())


def test_iterations_very_large_bf16(env):
    """fp16 features in pinned host memory, bf16 embeddings/weights/cache, bf16 MFMA linear. The node count (and
    with it edges, training subset and cache slots) is divided by 8 so that the table (47 GB instead of 375 GB)
    fits the host memory a job may pin here (94 GB was refused); row width, fan-outs, batch and cache fraction
    are those of the workload."""
    torch, B = env
    w = wl.WORKLOADS["very_large"].scaled(8)
    feat = None
    for fused in (True, False):   # the fused loader (what bench.py times) and the separate gather, on one table
        g = wl.make_graph(w)
        if feat is None:
            from fg_inputs import device as fdev
            feat = fdev.feature_table(w.seed, w.num_nodes, w.feat_dim, w.feat_dtype, w.feat_location)
        hits, worst = run_workload_parity(torch, w, 8 if fused else 3, check_numeric_every=3, sample_rows=20000, feat_table=feat,
                                          fused=fused, col_ids=fused)
        print(f"{w.name} (fused loader: {fused}): {hits} hits, worst rel err {worst:.3e}")
