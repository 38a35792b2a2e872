"""Decode rows whose scores hold a NaN or +inf: out and lse are NaN, whatever form the plan runs the step in, and every other row is what
it is without."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu

NARROW, WIDE, FP8_MATRIX, ONE_STREAM = 8, 16, 2, 4
PATHS, ITEMS, TILES = {}, {"tile_workgroups": 8}, {"tile_min_gflop": -1}     # the second: a setting that these plans have no use for


def attend(gpu, dp, f, q, **settings):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, q.shape[1], **settings)
    assert (hkv.hkv_decode_plan_num_paths(plan) > 0) == (settings == PATHS)
    assert (hkv.hkv_decode_plan_num_tile_items(plan) > 0) == ("tile_min_gflop" in settings)
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    ws, out = torch.empty(nb, dtype=torch.uint8, device="cuda"), torch.empty_like(q)
    lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
    hkv.attn_decode_plan_run(plan, q, 1.0 / np.sqrt(128.0), out, lse, ws, nb)
    torch.cuda.synchronize()
    hkv.hkv_decode_plan_destroy(plan)
    return out.float().cpu().numpy(), lse.cpu().numpy()


@pytest.mark.parametrize("kv_dtype, settings", [
    (wl.KV_BF16, PATHS), (wl.KV_BF16, ITEMS), (wl.KV_BF16, {"pack": 3}), (wl.KV_BF16, {"flags": NARROW}), (wl.KV_BF16, {"flags": WIDE}),
    (wl.KV_BF16, {"flags": NARROW, "shared_chunk": 64, "leaf_chunk": 16}), (wl.KV_BF16, TILES), (wl.KV_BF16, {**TILES, "flags": ONE_STREAM, "fused": -1}),
    (wl.KV_FP8_E4M3, PATHS), (wl.KV_FP8_E4M3, ITEMS), (wl.KV_FP8_E4M3, {"pack": 3}), (wl.KV_FP8_E4M3, {"flags": FP8_MATRIX}), (wl.KV_FP8_E4M3, TILES)])
@pytest.mark.parametrize("where", ["root", "first_block", "leaf", "on_the_root"])
def test_nan_and_infinite_scores(gpu, kv_dtype, settings, where):  # noqa: F811
    """where: one token of the shared node or of its first 32; every token of a leaf (nothing else is in its partial); every token of the
    shared node, with requests that end there (nothing else is in their rows)."""
    import torch
    n_req = 80 if "tile_min_gflop" in settings else 6
    parent, ntok, leaves = [-1] + [0] * n_req, [300] + [1 + 17 * r % 60 for r in range(n_req)], list(range(1, n_req + 1))
    leaves[4] = 0
    n_used = sum(-(-t // 16) for t in ntok)
    f = wl.make_forest(parent, ntok, leaves, np.random.default_rng(1).permutation(n_used).astype(np.int32))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    dp = gpu.DevicePool(n_used, 2, kv_dtype)
    q = torch.randn((n_req, 8, 128), device="cuda", generator=gen).bfloat16()
    q[:, :, 0] = 1.0
    kv = [tuple(torch.randn((t, 2, 128), device="cuda", generator=gen).bfloat16() for _ in range(2)) for t in ntok]

    def write(v, k):
        dp.write(f.node_pages[f.page_begin[v]: f.page_begin[v] + f.n_pages[v]], 0, k, kv[v][1])

    for v in range(len(ntok)):
        write(v, kv[v][0])
    clean, clean_l = attend(gpu, dp, f, q, **settings)
    assert np.isfinite(clean).all() and np.isfinite(clean_l).all()
    node, tokens, hit = {"root": (0, slice(70, 71), slice(None)), "first_block": (0, slice(9, 10), slice(None)), "leaf": (3, slice(None), slice(2, 3)),
                         "on_the_root": (0, slice(None), slice(None))}[where]
    for bad in (float("nan"),) + ((float("inf"),) if kv_dtype == wl.KV_BF16 else ()):
        if kv_dtype == wl.KV_FP8_E4M3:      # (a store turns a NaN into a number: the codes themselves, 0x7F is NaN)
            codes = dp.k.view(torch.uint8).view(n_used, 2, 2, 16, 64)     # block, head, dim / 64, slot, dim % 64
            for t in range(ntok[node])[tokens]:
                codes[int(f.node_pages[f.page_begin[node] + t // 16]), 1, 0, t % 16, 0] = 0x7F
        else:
            k = kv[node][0].clone()
            k[tokens, 1, 0] = bad
            write(node, k)
        got, got_l = attend(gpu, dp, f, q, **settings)
        assert np.isnan(got[hit, 4:]).all() and np.isnan(got_l[hit, 4:]).all(), (where, bad)
        rest = np.ones((n_req, 8), dtype=bool)
        rest[hit, 4:] = False
        assert np.array_equal(got[rest], clean[rest]) and np.array_equal(got_l[rest], clean_l[rest]), (where, bad)
    dp.close()
