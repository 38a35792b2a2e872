"""Suffix prefill of batches small enough to be split along their keys: one to a few requests over a long cached prefix, so that
a tile's key blocks go to several workgroups and a second kernel combines their results.  Segments that end inside the causal
part (rows that see nothing of one), ragged ends with NaN behind them, pages of several blocks, a dominant key inside one
segment (running-maximum path, counted once per tile), whole tiles in front of cut ones, segments longer than the window of page ids
in LDS, infinities and NaN, against the oracle or the same plan's whole tiles."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import LSE_ABS_FP8_PREFILL, both_pools, check_close, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def workload(hq, hk, prefix, new, kv_dtype=wl.KV_BF16, page_size=16, cls=wl.Workload):
    parent, ntok = [-1] + [0] * len(new), [prefix] + list(new)
    n_used = sum((t + page_size - 1) // page_size for t in ntok)
    pages = np.random.default_rng([prefix, *new]).permutation(n_used + 5).astype(np.int32)
    f = wl.make_forest(parent, ntok, list(range(1, len(new) + 1)), pages, page_size)
    return cls(name=f"{hq}_{hk}_{prefix}_{new}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=kv_dtype, num_pages=n_used + 5, seed=prefix + sum(new),
               forest=f, mode="prefill", q_len=np.asarray(new, dtype=np.int32))


def run(gpu, oracle, w, runs=1, whole_too=False):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    r = gpu.PrefillRunner(dp, w)
    segments = hkv.hkv_prefill_plan_segments(r.plan)
    assert (segments[:, 9] >= 0).any() and (segments[:, 9] < 0).any() == whole_too
    for _ in range(runs):
        r.out.fill_(0x7FC0)
        r.lse.fill_(float("nan"))
        r.run()
    torch.cuda.synchronize()
    got_o, got_l = gpu.bf16_tensor_to_f64(r.out), r.lse.cpu().numpy()
    fallback = hkv.hkv_prefill_plan_fallback_tiles(r.plan)
    n_tiles = len(hkv.hkv_prefill_plan_tiles(r.plan))
    r.close()
    dp.close()
    check_close(got_o, exp_o, w.name)
    check_lse(got_l, exp_l, w.name, tol=LSE_ABS_FP8_PREFILL if w.kv_dtype == wl.KV_FP8_E4M3 else 2e-3 + 1e-6 * np.abs(exp_l).max())
    return fallback, n_tiles


@pytest.mark.parametrize("hq, hk, prefix, new", [
    (8, 2, 2048, (1,)), (8, 2, 2048, (64,)), (8, 2, 2064, (65, 3)), (8, 2, 4112, (200,)),
    (2, 2, 1040, (255,)), (2, 2, 1040, (257, 300)), (4, 2, 1104, (700,)),       # 256 resp. 128 tokens per tile: segments cut the diagonal
    (5, 1, 1500 // 16 * 16, (51, 52, 103)), (16, 1, 1600, (16, 17, 1)), (3, 3, 1024, (86, 400)),
    (8, 8, 1008, (256 * 9 + 1,)),
])
def test_split_prefill(gpu, oracle, hq, hk, prefix, new):  # noqa: F811
    assert run(gpu, oracle, workload(hq, hk, prefix, new), runs=2)[0] == 0


@pytest.mark.parametrize("hq, hk, prefix, new", [(32, 8, 2048, (256, 300, 350, 400, 450, 512)), (16, 8, 2064, (769, 700, 660, 641, 640, 600, 600))])
def test_whole_tiles_in_front_of_cut_ones(gpu, oracle, hq, hk, prefix, new):  # noqa: F811
    """A few more tiles per head than workers: every worker runs a whole tile, then its share of the others' key blocks."""
    run(gpu, oracle, workload(hq, hk, prefix, new), whole_too=True)


@pytest.mark.parametrize("kv_dtype, page_size", [(wl.KV_FP8_E4M3, 16), (wl.KV_BF16, 64), (wl.KV_FP8_E4M3, 32)])
def test_split_prefill_pools_and_pages(gpu, oracle, kv_dtype, page_size):  # noqa: F811
    run(gpu, oracle, workload(8, 2, 2048, (77, 130), kv_dtype, page_size))


class Loud(wl.Workload):
    """One token in the middle of the prefix whose key dwarfs the others."""

    def node_kv(self, node):
        k, v = super().node_kv(node)
        if node == 0:
            k = wl.bf16_bits_to_f32(k).copy()
            k[1500] = 60.0 * np.sign(k[1500])
            k = wl.f32_to_bf16_bits(k)
        return k, v


def test_split_prefill_running_maximum(gpu, oracle):  # noqa: F811
    fallback, n_tiles = run(gpu, oracle, workload(8, 2, 3072, (130,), cls=Loud))
    assert 0 < fallback <= n_tiles


def test_split_prefill_under_graph_replay(gpu):  # noqa: F811
    """Two kernels over the partials in the caller's workspace: every replay gives the eager result's bits."""
    import torch
    w = workload(8, 2, 2048, (130, 40))
    dp = gpu.DevicePool(w.num_pages, w.num_kv_heads, w.kv_dtype)
    dp.fill_from(w)
    r = gpu.PrefillRunner(dp, w)
    r.run()
    torch.cuda.synchronize()
    ref_o, ref_l = r.out.clone(), r.lse.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        r.run()
    for _ in range(3):
        r.out.fill_(7)
        r.lse.fill_(3.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(r.out, ref_o) and torch.equal(r.lse, ref_l)
        r.run()                                        # eager work on the same partials between replays
    del g
    r.close()
    dp.close()


@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
def test_room_for_partials_is_the_callers(gpu, oracle, kv_dtype):  # noqa: F811
    """With the whole workspace the tiles are split and nothing behind it is touched; with an fp8 pool's pages only, with none, or
    with one that is not aligned (bf16 pools ignored it before there were partials) they stay whole and the results agree."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    w = workload(8, 2, 2048, (130, 40), kv_dtype)
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    r = gpu.PrefillRunner(dp, w)
    need = hkv.hkv_prefill_plan_workspace_bytes(r.plan)
    blocks = sum(int(n) for n in w.forest.n_pages)
    pages = blocks * 2 * 8192 if kv_dtype == wl.KV_FP8_E4M3 else 0
    assert need > pages
    ws = torch.full((need + 512,), 0x5A, dtype=torch.uint8, device="cuda")

    def run_with(buffer, nbytes):
        r.out.fill_(0x7FC0)
        r.lse.fill_(float("nan"))
        hkv.attn_prefill_plan_run(r.plan, r.q, r.scale, r.out, r.lse, None, buffer, nbytes)
        torch.cuda.synchronize()
        check_close(gpu.bf16_tensor_to_f64(r.out), exp_o, w.name)
        check_lse(r.lse.cpu().numpy(), exp_l, w.name, tol=LSE_ABS_FP8_PREFILL)
        return r.out.clone(), r.lse.clone()

    split = run_with(ws, need)
    assert (ws[need:] == 0x5A).all() and (ws[pages:need] != 0x5A).any()
    ws[pages:] = 0x5A
    whole = run_with(ws, need - 1)
    assert (ws[pages:] == 0x5A).all()
    assert not torch.equal(whole[1], split[1])          # another order of the sums
    others = [run_with(ws, pages)] if pages else [run_with(None, 0), run_with(ws[1:], need + 511)]
    for o, ls in others:
        assert torch.equal(o, whole[0]) and torch.equal(ls, whole[1])
    assert (ws[pages:] == 0x5A).all()
    r.close()
    dp.close()


@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
def test_one_shot_calls_on_two_streams(gpu, kv_dtype):  # noqa: F811
    """The one-shot form keeps its plan in the pool.  Calls over the same tables on two streams, each with its own queries, results
    and workspace, share nothing that either writes: both give the bits they give alone."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    w = workload(8, 2, 4096, (200, 150), kv_dtype)
    dp = gpu.DevicePool(w.num_pages, w.num_kv_heads, w.kv_dtype)
    dp.fill_from(w)
    r = gpu.PrefillRunner(dp, w)
    side = [torch.cuda.Stream(), torch.cuda.Stream()]
    q = [r.q, r.q.flip(0).contiguous()]
    out, lse = [torch.zeros_like(r.out) for _ in q], [torch.zeros_like(r.lse) for _ in q]
    ws = [torch.empty(r.ws_bytes, dtype=torch.uint8, device="cuda") for _ in q]

    def call(i, stream):
        hkv.attn_prefill_with_prefix(dp.handle, q[i], r.cu_q, r.block_table, r.kv_len, w.num_q_heads, r.scale, out[i], lse[i], ws[i], r.ws_bytes,
                                     stream)

    alone = []
    for i in range(2):
        call(i, side[i].cuda_stream)
        torch.cuda.synchronize()
        alone.append((out[i].clone(), lse[i].clone()))
    assert not torch.equal(alone[0][0], alone[1][0])
    for _ in range(20):
        for i in range(2):
            out[i].fill_(7)
            lse[i].fill_(7.0)
        torch.cuda.synchronize()
        for _ in range(4):
            for i in range(2):
                call(i, side[i].cuda_stream)
        torch.cuda.synchronize()
        for i in range(2):
            assert torch.equal(out[i], alone[i][0]) and torch.equal(lse[i], alone[i][1])
    r.close()
    dp.close()


def test_segment_that_begins_with_keys_of_score_minus_infinity(gpu):  # noqa: F811
    """The first 32 keys of a segment score -inf and all others about -300 powers of two: a segment has no reference from its
    first scores then, and one that is not its rows' own would make all their weights underflow."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    prefix, new, hq, hk = 2048, 64, 8, 2
    w = workload(hq, hk, prefix, (new,))
    dp = gpu.DevicePool(w.num_pages, hk, w.kv_dtype)
    r = gpu.PrefillRunner(dp, w)
    seg = hkv.hkv_prefill_plan_segments(r.plan)
    first = prefix - seg[(seg[:, 3] == 0) & (seg[:, 5] < prefix)][1, 5]          # of some segment behind the first one
    assert 0 < first < prefix - 32
    rng = np.random.default_rng(9)
    bits, back = wl.f32_to_bf16_bits, wl.bf16_bits_to_f32
    K = rng.standard_normal((prefix + new, hk, 128)).astype(np.float32)
    K[:, :, 0], K[:, :, 1] = 0.0, -300.0
    K[first: first + 32, :, 0] = -np.inf
    V = rng.standard_normal((prefix + new, hk, 128)).astype(np.float32)
    q = 0.1 * rng.standard_normal((new, hq, 128)).astype(np.float32)
    q[:, :, :2] = 1.0
    K, V, q = back(bits(K)), back(bits(V)), back(bits(q))
    for node, part in ((0, slice(0, prefix)), (1, slice(prefix, prefix + new))):
        f = w.forest
        pages = f.node_pages[f.page_begin[node]: f.page_begin[node] + f.n_pages[node]]
        dp.write(pages, 0, gpu.to_device_bits(bits(K[part])), gpu.to_device_bits(bits(V[part])))
    out = torch.zeros((new, hq, 128), dtype=torch.int16, device="cuda")
    lse = torch.zeros((new, hq), dtype=torch.float32, device="cuda")
    scale = float(np.log(2.0))
    hkv.attn_prefill_plan_run(r.plan, gpu.to_device_bits(bits(q)), scale, out, lse, None, r.ws, r.ws_bytes)
    torch.cuda.synchronize()
    exp_o, exp_l = np.zeros((new, hq, 128)), np.zeros((new, hq))
    keep = np.ones(prefix + new, dtype=bool)
    keep[first: first + 32] = False
    for i in range(new):
        seen = keep & (np.arange(prefix + new) <= prefix + i)
        for h in range(hq):
            s = K[seen, h // (hq // hk)].astype(np.float64) @ q[i, h].astype(np.float64) * scale
            exp_l[i, h] = s.max() + np.log(np.exp(s - s.max()).sum())
            exp_o[i, h] = np.exp(s - exp_l[i, h]) @ V[seen, h // (hq // hk)]
    check_close(gpu.bf16_tensor_to_f64(out), exp_o, "-inf at a segment's start")
    check_lse(lse.cpu().numpy(), exp_l, "-inf at a segment's start", tol=2e-3 + 1e-6 * np.abs(exp_l).max())
    r.close()
    dp.close()


def run_form(gpu, r, ws):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    r.out.fill_(0x7FC0)
    r.lse.fill_(float("nan"))
    hkv.attn_prefill_plan_run(r.plan, r.q, r.scale, r.out, r.lse, None, ws, r.ws_bytes if ws is not None else 0)
    torch.cuda.synchronize()
    return gpu.bf16_tensor_to_f64(r.out), r.lse.cpu().numpy()


@pytest.mark.parametrize("late_key", [False, True])
def test_segments_longer_than_the_page_id_window(gpu, late_key):  # noqa: F811
    """24 requests over 65 536 cached tokens, 8 heads: segments of up to 773 key blocks, the window holds the ids of 512.  late_key: a
    dominant key behind the refill point of the longest segment, so that the running-maximum loop refills it too.  Whole tiles (1026
    blocks, refilled as well) and split ones against attention in float64 for a request's first and last tokens."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    root, n_req, hq = 65536, 24, 8
    n_pages = root // 16 + 7 * n_req
    f = wl.make_forest([-1] + [0] * n_req, [root] + [100] * n_req, list(range(1, n_req + 1)),
                       np.random.default_rng(2).permutation(n_pages).astype(np.int32))
    w = wl.Workload(name="long_segments", num_q_heads=hq, num_kv_heads=hq, kv_dtype=wl.KV_BF16, num_pages=n_pages, seed=3, forest=f, mode="prefill",
                    q_len=np.full(n_req, 100, dtype=np.int32))
    dp = gpu.DevicePool(n_pages, hq, wl.KV_BF16)
    r = gpu.PrefillRunner(dp, w, random_q=True)
    seg = hkv.hkv_prefill_plan_segments(r.plan)
    longest = seg[np.argmax(seg[:, 8])]
    assert longest[8] > 64 * 520
    at = root - longest[5] + 64 * 515                       # (the tile's prefix is the root; moved to the segment's first key)
    assert at < root
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    K = torch.randn((root + n_req * 100, hq, 128), device="cuda", generator=gen).to(torch.bfloat16)
    V = torch.randn((root + n_req * 100, hq, 128), device="cuda", generator=gen).to(torch.bfloat16)
    if late_key:
        K[at] = 0.0
        K[at, :, 0] = 300.0
        r.q.view(torch.bfloat16)[:, :, 0] = 4.0             # a score of 1200 * scale = 106, 100 above the others
    for v in range(n_req + 1):
        part = slice(0, root) if v == 0 else slice(root + 100 * (v - 1), root + 100 * v)
        dp.write(f.node_pages[f.page_begin[v]: f.page_begin[v] + f.n_pages[v]], 0, K[part].view(torch.int16), V[part].view(torch.int16))
    q = r.q.view(torch.bfloat16).double()
    req = int(longest[0])
    rows, exp_o, exp_l = [100 * req + i for i in (0, 1, 50, 99)], [], []
    for row in rows:
        own = slice(root + 100 * req, root + row + 1)
        k, v = (torch.cat([x[:root], x[own]]).double().permute(1, 2, 0).contiguous() for x in (K, V))
        s = (q[row][:, None, :] @ k)[:, 0] * r.scale
        l = torch.logsumexp(s, dim=1)
        exp_l.append(l.cpu().numpy())
        exp_o.append((v @ torch.exp(s - l[:, None])[:, :, None])[:, :, 0].cpu().numpy())
    exp_o, exp_l = np.asarray(exp_o), np.asarray(exp_l)
    whole_o, whole_l = run_form(gpu, r, None)
    split_o, split_l = run_form(gpu, r, r.ws)
    fallback = hkv.hkv_prefill_plan_fallback_tiles(r.plan)
    assert fallback == (2 * len(hkv.hkv_prefill_plan_tiles(r.plan)) if late_key else 0)
    for o, ls in ((whole_o, whole_l), (split_o, split_l)):
        check_close(o[rows], exp_o, "long segments")
        check_lse(ls[rows], exp_l, "long segments", tol=2e-3 + 1e-6 * np.abs(exp_l).max())
    check_close(split_o, whole_o, "split against whole")
    r.close()
    dp.close()


def test_infinities_and_nan_show_where_whole_tiles_show_them(gpu):  # noqa: F811
    """Infinite and NaN values and keys inside the prefix and inside the causal part: split and whole tiles agree on which results
    are finite, and on those."""
    import torch
    w = workload(8, 2, 2048, (130, 40))
    f = w.forest
    dp = gpu.DevicePool(w.num_pages, 2, wl.KV_BF16)
    bits, back = wl.f32_to_bf16_bits, wl.bf16_bits_to_f32
    for trial in range(6):
        for v in range(f.n_nodes):
            K, V = (back(x).copy() for x in w.node_kv(v))
            if trial == 0 and v == 0:
                V[700, 0, 3], V[1500, 1, 4] = np.inf, -np.inf
            if trial == 1 and v == 0:
                K[64, 0, 5] = np.nan
            if trial == 2 and v == 0:
                K[1990, 1, 5] = np.inf
            if trial == 3 and v == 1:
                V[100, 0, 6] = np.nan
            if trial == 4 and v == 1:
                K[64, 0, 7] = -np.inf
            if trial == 5 and v == 2:
                K[39, 1, 0] = np.nan
            dp.write(f.node_pages[f.page_begin[v]: f.page_begin[v] + f.n_pages[v]], 0, gpu.to_device_bits(bits(K)), gpu.to_device_bits(bits(V)))
        r = gpu.PrefillRunner(dp, w)
        (whole_o, whole_l), (split_o, split_l) = run_form(gpu, r, None), run_form(gpu, r, r.ws)
        assert not np.isfinite(whole_o).all() and np.isfinite(whole_o).any()
        assert np.array_equal(np.isfinite(whole_o), np.isfinite(split_o)) and np.array_equal(np.isfinite(whole_l), np.isfinite(split_l)), trial
        fin, fin_l = np.isfinite(whole_o), np.isfinite(whole_l)
        check_close(split_o[fin], whole_o[fin], f"trial {trial}")
        check_lse(split_l[fin_l], whole_l[fin_l], f"trial {trial}")
        r.close()
    torch.cuda.synchronize()
    dp.close()
