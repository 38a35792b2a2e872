"""Suffix prefill of batches small enough to be split along their keys: one to a few requests over a long cached prefix, so that
a tile's key blocks go to several workgroups and a second kernel combines their results.  Segments that end inside the causal
part (rows that see nothing of one), ragged ends with NaN behind them, pages of several blocks, a dominant key inside one
segment (running-maximum path, counted once per tile), whole tiles in front of cut ones, against the oracle."""
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


def run(gpu, oracle, w, runs=1):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    r = gpu.PrefillRunner(dp, w)
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
    """Two kernels over the plan's own partials: every replay gives the eager result's bits."""
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
