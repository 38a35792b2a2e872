"""Small decode steps, which run whole root-to-leaf paths in one launch, and the same plans as items: the edges of blocks, steps and
wavefronts, nodes that end inside a block anywhere on a path, empty ones, requests on inner nodes and several on one leaf, drafted
tokens, rows given by the caller, scores of -inf and NaN, against the oracle."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import both_pools, check_close, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu

FORMS = [{}, {"tile_workgroups": 8}]     # the library's choice; a planner setting (one that these plans have no use for): items
FORESTS = {
    "one_token": ([-1], [1], [0], 1),
    "block_edges": ([-1, 0, 0, 0], [16, 15, 16, 17], [1, 2, 3], 1),
    "holes": ([-1, 0, 1, 1, 0, 4], [13, 30, 1, 47, 33, 5], [2, 3, 5, 4, 0, 2, 2], 1),     # inner nodes, three requests on one leaf
    "empty_nodes": ([-1, 0, 1, 0, -1, 4], [0, 40, 0, 7, 0, 0], [2, 3, 5, 1], 1),          # request 2 sees no token at all
    "eight_wavefronts": ([-1] + [0] * 5, [255, 1, 2, 33, 257, 300], [1, 2, 3, 4, 5], 1),
    "four_wavefronts": ([-1] + [0] * 66, [67] + [1 + 7 * i % 60 for i in range(66)], list(range(1, 67)), 1),
    "drafted": ([-1, 0, 0], [77, 9, 40], [1, 2], 8),
    "drafted_tree": ([-1, 0, 0], [64, 21, 50], [1, 2], 21),
}


def masks(T, n_req):
    if T <= 16:
        return np.tile(np.asarray([(1 << (t + 1)) - 1 for t in range(T)], dtype=np.uint64), n_req)
    one = [1 << t | (0 if t < 3 else 1 << (t % 3)) for t in range(T)]      # children of three drafted tokens
    return np.tile(np.asarray(one, dtype=np.uint64), n_req)


@pytest.mark.parametrize("settings", FORMS)
@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("hq, hk", [(8, 2), (16, 1), (5, 5), (40, 8)])
def test_forests(gpu, oracle, kv_dtype, hq, hk, settings):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    for name, (parent, ntok, leaves, T) in FORESTS.items():
        n_used = sum((t + 15) // 16 for t in ntok)
        pages = np.random.default_rng([n_used, hq]).permutation(n_used + 3).astype(np.int32)
        f = wl.make_forest(parent, ntok, leaves, pages)
        w = wl.Workload(name=name, num_q_heads=hq, num_kv_heads=hk, kv_dtype=kv_dtype, num_pages=n_used + 3, seed=hq + n_used, forest=f, mode="decode")
        hp, dp = both_pools(gpu, oracle, w)
        rng = np.random.default_rng(w.seed)
        n = f.n_req * T
        q = wl.f32_to_bf16_bits(rng.standard_normal((n, hq, 128)).astype(np.float32))
        seen = masks(T, f.n_req) if T > 1 else None
        exp_o, exp_l = oracle.attn_decode_tree(hp, q, f.nodes, f.node_pages, np.repeat(f.req_leaf, T), float(w.scale),
                                               tail_len=T if T > 1 else 0, tail_mask=seen)
        to = rng.permutation(n + 4)[:n].astype(np.int32)                  # row r of the plan is row to[r] of q, out and lse
        q_rows = np.zeros((n + 4, hq, 128), dtype=q.dtype)
        q_rows[to] = q
        plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, hq, tokens_per_req=T,
                                             visible=seen if T > 16 else None, q_rows=to, **settings)
        per_path = max(1, 16 // (hq // hk))
        on_leaf = np.bincount(np.repeat(f.req_leaf, T))
        assert hkv.hkv_decode_plan_num_paths(plan) == (0 if settings else int(np.sum(-(-on_leaf // per_path)))), name
        nb = hkv.hkv_decode_plan_workspace_bytes(plan)
        ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
        out = torch.full((n + 4, hq, 128), 7, dtype=torch.int16, device="cuda")
        lse = torch.full((n + 4, hq), 7.0, dtype=torch.float32, device="cuda")
        hkv.attn_decode_plan_run(plan, gpu.to_device_bits(q_rows), float(w.scale), out, lse, ws, nb)
        torch.cuda.synchronize()
        hkv.hkv_decode_plan_destroy(plan)
        dp.close()
        what = f"{name} {hq}/{hk} dtype {kv_dtype} {settings}"
        check_close(gpu.bf16_tensor_to_f64(out)[to], exp_o, what)
        got, none = lse.cpu().numpy()[to], np.isneginf(exp_l)
        assert np.array_equal(np.isneginf(got), none), what
        check_lse(np.where(none, 0, got), np.where(none, 0, exp_l), what)
        rest = np.setdiff1d(np.arange(n + 4), to)
        assert (out.cpu().numpy()[rest] == 7).all() and (lse.cpu().numpy()[rest] == 7).all(), what


@pytest.mark.parametrize("quiet", [range(0, 31), range(0, 300), range(5, 300)])
def test_scores_of_minus_infinity_and_nan(gpu, oracle, quiet):  # noqa: F811
    """Tokens `quiet` of the root score -inf (a wavefront's only ones, all of some wavefronts'): the rest is plain attention.  A NaN
    among the keys of one head gives NaN in that head's rows below it, and only there."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    parent, ntok, leaves = [-1, 0, 0, 0], [300, 20, 1, 33], [1, 2, 3]
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, leaves, np.arange(n_used, dtype=np.int32))
    w = wl.Workload(name="quiet", num_q_heads=8, num_kv_heads=2, kv_dtype=wl.KV_BF16, num_pages=n_used, seed=3, forest=f, mode="decode")
    bits, back = wl.f32_to_bf16_bits, wl.bf16_bits_to_f32
    q = back(w.q()).copy()
    q[:, :, 0] = 1.0
    for nan in (False, True):
        dp = gpu.DevicePool(n_used, 2, wl.KV_BF16)
        kv = []
        for v in range(f.n_nodes):
            K, V = (back(x).copy() for x in w.node_kv(v))
            K[:, :, 0] = 0.0
            if v == 0:
                K[list(quiet), :, 0] = -np.inf
            if v == 3 and nan:
                K[11, 1, 5] = np.nan
            kv.append((K, V))
            dp.write(f.node_pages[f.page_begin[v]: f.page_begin[v] + f.n_pages[v]], 0, gpu.to_device_bits(bits(K)), gpu.to_device_bits(bits(V)))
        plan = hkv.hkv_decode_plan_create(dp.handle, f.nodes, f.node_pages, f.req_leaf, 8)
        assert hkv.hkv_decode_plan_num_paths(plan) == 3
        nb = hkv.hkv_decode_plan_workspace_bytes(plan)
        ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
        out = torch.zeros((3, 8, 128), dtype=torch.int16, device="cuda")
        lse = torch.zeros((3, 8), dtype=torch.float32, device="cuda")
        hkv.attn_decode_plan_run(plan, gpu.to_device_bits(bits(q)), float(w.scale), out, lse, ws, nb)
        torch.cuda.synchronize()
        hkv.hkv_decode_plan_destroy(plan)
        dp.close()
        got, got_l = gpu.bf16_tensor_to_f64(out), lse.cpu().numpy()
        for r, leaf in enumerate(leaves):
            K, V = (np.concatenate([kv[0][i], kv[leaf][i]]).astype(np.float64) for i in range(2))
            for h in range(8):
                if nan and leaf == 3 and h >= 4:
                    assert np.isnan(got[r, h]).all() and np.isnan(got_l[r, h])
                    continue
                s = (K[:, h // 4, 1:] @ q[r, h, 1:].astype(np.float64) + K[:, h // 4, 0]) * float(w.scale)
                e = np.exp(s - s.max())
                check_close(got[r, h], e @ V[:, h // 4] / e.sum(), f"{r} {h}")
                check_lse(got_l[r, h], s.max() + np.log(e.sum()), f"{r} {h}")


@pytest.mark.parametrize("spread", [0, 12, 39, 44, 60])
def test_scales_of_fp8_blocks_far_apart(gpu, oracle, spread):  # noqa: F811
    """V blocks whose scales differ by up to 2^(2 * spread), within and beyond the range in which they ride in the exponents: every row
    against the oracle in units of its own largest value (a row holds the few blocks of the largest scale and their share)."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    parent, ntok, leaves = [-1, 0, 0], [200, 33, 90], [1, 2]
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, leaves, np.arange(n_used, dtype=np.int32))

    class Scaled(wl.Workload):
        def node_kv(self, node):
            k, v = super().node_kv(node)
            e = np.random.default_rng([node, spread]).integers(-spread, spread + 1, size=(len(v) + 15) // 16)
            return k, wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(v) * np.exp2(e.astype(np.float32)).repeat(16)[: len(v), None, None])

    w = Scaled(name=f"scales{spread}", num_q_heads=8, num_kv_heads=2, kv_dtype=wl.KV_FP8_E4M3, num_pages=n_used, seed=9, forest=f, mode="decode")
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    plan = hkv.hkv_decode_plan_create(dp.handle, f.nodes, f.node_pages, f.req_leaf, 8)
    assert hkv.hkv_decode_plan_num_paths(plan) == 2
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
    out = torch.zeros((2, 8, 128), dtype=torch.int16, device="cuda")
    lse = torch.zeros((2, 8), dtype=torch.float32, device="cuda")
    hkv.attn_decode_plan_run(plan, gpu.to_device_bits(w.q()), float(w.scale), out, lse, ws, nb)
    torch.cuda.synchronize()
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()
    top = np.abs(exp_o).max(axis=2, keepdims=True)
    check_close(gpu.bf16_tensor_to_f64(out) / top, exp_o / top, w.name)
    check_lse(lse.cpu().numpy(), exp_l, w.name)
