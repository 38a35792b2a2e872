"""Decode items shared by 17 to 64 query rows, in both forms (two 32-row tiles x two token halves per workgroup; for bf16 pools
also four 16-row tiles): the edges of row tiles, of token halves and of the 64-token block, scores that rise far above the first
block's (where the softmax reference moves), rows that see nothing of a chunk, scores of -inf and NaN, and the split of more than 64
rows into equal groups, against the oracle."""
import dataclasses

import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import both_pools, check_close, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@dataclasses.dataclass
class Rising(wl.Workload):
    """Keys that grow with the token: the largest scores of a node lie in its last blocks."""
    gain: float = 1.0

    def node_kv(self, node):
        k, v = super().node_kv(node)
        up = (1.0 + self.gain * np.arange(k.shape[0]) / max(1, k.shape[0])).astype(np.float32)[:, None, None]
        return wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(k) * up), v


def workload(kv_dtype, hq, hk, n_req, root, gain=0.0):
    parent, ntok = [-1] + [0] * n_req, [root] + [1 + 3 * r % 40 for r in range(n_req)]
    n_used = sum((t + 15) // 16 for t in ntok)
    pages = np.random.default_rng([n_req, root]).permutation(n_used + 5).astype(np.int32)
    f = wl.make_forest(parent, ntok, list(range(1, n_req + 1)), pages)
    return Rising(name=f"root{root}_x{n_req}_{hq}_{hk}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=kv_dtype, num_pages=n_used + 5,
                  seed=root + n_req, forest=f, mode="decode", gain=gain)


def run(gpu, oracle, w, T=1, tiles=(False, False), **settings):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    hp, dp = both_pools(gpu, oracle, w)
    f = w.forest
    q = wl.f32_to_bf16_bits(np.random.default_rng(w.seed).standard_normal((f.n_req * T, w.num_q_heads, 128)).astype(np.float32))
    masks = np.tile(np.asarray([(1 << (t + 1)) - 1 for t in range(T)], dtype=np.uint64), f.n_req)
    if not any(settings.values()):
        settings = {"tile_workgroups": 8}      # fp8: items, not whole paths (a setting that these plans have no use for)
    exp_o, exp_l = oracle.attn_decode_tree(hp, q, f.nodes, f.node_pages, np.repeat(f.req_leaf, T), float(w.scale),
                                           tail_len=T if T > 1 else 0, tail_mask=masks if T > 1 else None)
    plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, w.num_q_heads, tokens_per_req=T,
                                         visible=masks if T > 16 else None, **settings)
    items = hkv.hkv_decode_plan_items(plan)
    G = w.num_q_heads // w.num_kv_heads
    n_tiles, fused = hkv.hkv_decode_plan_num_tile_items(plan), bool(hkv.hkv_decode_plan_is_fused(plan))
    assert (n_tiles > 0, fused) == tiles and hkv.hkv_decode_plan_num_paths(plan) == 0
    if not n_tiles:
        assert (items[:, 4] * G > 16).any() and (items[:, 4] * G <= 64).all()
        if w.kv_dtype == wl.KV_FP8_E4M3 or "flags" in settings:          # (bf16 without a flag: as the library estimates)
            assert hkv.hkv_decode_plan_has_wide_tiles(plan) == (settings.get("flags", 0) != hkv.PLAN_NARROW_TILES)
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
    out = torch.zeros((f.n_req * T, w.num_q_heads, 128), dtype=torch.int16, device="cuda")
    lse = torch.zeros((f.n_req * T, w.num_q_heads), dtype=torch.float32, device="cuda")
    hkv.attn_decode_plan_run(plan, gpu.to_device_bits(q), float(w.scale), out, lse, ws, nb)
    torch.cuda.synchronize()
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()
    check_close(gpu.bf16_tensor_to_f64(out), exp_o, w.name)
    check_lse(lse.cpu().numpy(), exp_l, w.name)


NARROW, WIDE = 8, 16                   # HKV_PLAN_NARROW_TILES: 16-row tiles, HKV_PLAN_WIDE_TILES: 32-row tiles
FORMS = [(wl.KV_BF16, WIDE), (wl.KV_FP8_E4M3, 0), (wl.KV_BF16, NARROW)]


@pytest.mark.parametrize("kv_dtype, flags", FORMS)
@pytest.mark.parametrize("hq, hk, n_req", [(9, 1, 2), (8, 2, 5), (8, 2, 8), (11, 1, 3), (16, 2, 8), (10, 2, 13), (4, 1, 17), (8, 1, 25)])
def test_row_tiles_and_token_edges(gpu, oracle, kv_dtype, flags, hq, hk, n_req):  # noqa: F811
    for root in (1, 16, 17, 31, 33, 64, 65, 96, 97, 130, 700):
        run(gpu, oracle, workload(kv_dtype, hq, hk, n_req, root), flags=flags)


@pytest.mark.parametrize("kv_dtype, flags", FORMS)
@pytest.mark.parametrize("settings", [{}, {"shared_chunk": 64}, {"shared_chunk": 2048, "stages": 4}, {"shared_chunk": 2048, "stages": 5},
                                      {"shared_chunk": 2048, "stages": 3}])       # 3: four stages for 32-row tiles, three for 16-row tiles
def test_rising_scores_and_ring_sizes(gpu, oracle, kv_dtype, flags, settings):  # noqa: F811
    run(gpu, oracle, workload(kv_dtype, 8, 2, 16, 2048 + 33, gain=15.0), flags=flags, **settings)


@pytest.mark.parametrize("kv_dtype, flags", FORMS)
@pytest.mark.parametrize("T, leaf_chunk", [(8, 0), (16, 16), (40, 32)])
def test_drafted_rows_of_one_leaf(gpu, oracle, kv_dtype, flags, T, leaf_chunk):  # noqa: F811
    """T x 4 rows of one leaf: causal limits inside the item, and (short chunks) rows that see nothing of one."""
    parent, ntok = [-1, 0, 0], [128, T + 37, T]
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, [1, 2], np.random.default_rng(T).permutation(n_used + 3).astype(np.int32))
    w = wl.Workload(name=f"draft{T}", num_q_heads=8, num_kv_heads=2, kv_dtype=kv_dtype, num_pages=n_used + 3, seed=T, forest=f, mode="decode")
    run(gpu, oracle, w, T, flags=flags, **({"leaf_chunk": leaf_chunk, "shared_chunk": leaf_chunk} if leaf_chunk else {}))


@pytest.mark.parametrize("flags", [WIDE, NARROW])
@pytest.mark.parametrize("quiet", [range(0, 64), range(32, 160), range(0, 400), range(7, 400)])
def test_scores_of_minus_infinity_and_nan(gpu, oracle, flags, quiet):  # noqa: F811
    """Tokens `quiet` of the root score -inf (whole blocks, a wavefront's first ones, the whole item): the rest is plain attention.
    A NaN among the keys of one head stays with that head."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    w = workload(wl.KV_BF16, 8, 2, 8, 400)
    f, n_req = w.forest, w.forest.n_req
    dp = gpu.DevicePool(w.num_pages, 2, wl.KV_BF16)
    bits, back = wl.f32_to_bf16_bits, wl.bf16_bits_to_f32
    q = back(w.q()).copy()
    q[:, :, 0] = 1.0
    kv = []
    for v in range(f.n_nodes):
        K, V = (back(x).copy() for x in w.node_kv(v))
        K[:, :, 0] = 0.0
        if v == 0:
            K[list(quiet), :, 0] = -np.inf
        kv.append((K, V))
        dp.write(f.node_pages[f.page_begin[v]: f.page_begin[v] + f.n_pages[v]], 0, gpu.to_device_bits(bits(K)), gpu.to_device_bits(bits(V)))
    plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, 8, flags)
    assert hkv.hkv_decode_plan_has_wide_tiles(plan) == (flags == WIDE)
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    out = torch.zeros((n_req, 8, 128), dtype=torch.int16, device="cuda")
    lse = torch.zeros((n_req, 8), dtype=torch.float32, device="cuda")

    def step():
        hkv.attn_decode_plan_run(plan, gpu.to_device_bits(bits(q)), float(w.scale), out, lse, ws, nb)
        torch.cuda.synchronize()
        return gpu.bf16_tensor_to_f64(out), lse.cpu().numpy()

    exp_o, exp_l = np.zeros((n_req, 8, 128)), np.zeros((n_req, 8))
    for r in range(n_req):
        keep = [t for t in range(400) if t not in quiet]
        K, V = (np.concatenate([kv[0][i][keep], kv[f.req_leaf[r]][i]]).astype(np.float64) for i in (0, 1))
        for h in range(8):
            s = K[:, h // 4] @ q[r, h].astype(np.float64) * float(w.scale)
            exp_l[r, h] = s.max() + np.log(np.exp(s - s.max()).sum())
            exp_o[r, h] = np.exp(s - exp_l[r, h]) @ V[:, h // 4]
    got_o, got_l = step()
    check_close(got_o, exp_o, "-inf scores")
    check_lse(got_l, exp_l, "-inf scores")
    K = kv[0][0]
    K[70, 0, 5] = np.nan
    dp.write(f.node_pages[f.page_begin[0]: f.page_begin[0] + f.n_pages[0]], 0, gpu.to_device_bits(bits(K)), gpu.to_device_bits(bits(kv[0][1])))
    nan_o, nan_l = step()
    assert np.array_equal(nan_o[:, 4:], got_o[:, 4:]) and np.array_equal(nan_l[:, 4:], got_l[:, 4:])
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()


@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("T, n_req", [(8, 48), (4, 84)])
def test_tiles_above_drafted_rows(gpu, oracle, kv_dtype, T, n_req):  # noqa: F811
    """Several query tokens per request over a root shared by more than 256 rows: the root goes to the 256-row tile, the
    leaves with their causal limits to the other items' kernel behind it; not beside leaves of 16 rows."""
    parent, ntok = [-1] + [0] * n_req, [1040] + [T + 5 * r % 50 for r in range(n_req)]
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(1, n_req + 1)), np.random.default_rng(T).permutation(n_used + 3).astype(np.int32))
    w = wl.Workload(name=f"tiles{T}", num_q_heads=8, num_kv_heads=2, kv_dtype=kv_dtype, num_pages=n_used + 3, seed=T, forest=f, mode="decode")
    run(gpu, oracle, w, T, tiles=(T == 8, False), tile_min_gflop=1)


def weight_of_one_key(gpu, n_req, T, root, where, tiles=False, hq=8, hk=2, **settings):  # noqa: F811
    """Rows over `root` shared tokens (bf16) in which one key, token `where`, scores 0.3 to 7.7 powers of two above two keys of
    the first block whose values are zero; nothing else has weight.  Returns each row's relative error of that key's weight,
    the factor by which its result is the key's value."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    parent, ntok = [-1] + [0] * n_req, [root] + [T + r % 3 for r in range(n_req)]
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(1, n_req + 1)), np.random.default_rng(root).permutation(n_used).astype(np.int32))
    rng = np.random.default_rng([n_req, T, root])
    bits, back = wl.f32_to_bf16_bits, wl.bf16_bits_to_f32
    dp = gpu.DevicePool(n_used, hk, wl.KV_BF16)
    for v in range(len(ntok)):
        K, V = np.zeros((ntok[v], hk, 128), dtype=np.float32), np.zeros((ntok[v], hk, 128), dtype=np.float32)
        K[:, :, 1] = -60.0
        if v == 0:
            K[[0, 40, where], :, 1] = 0.0
            K[where, :, 0] = 1.0
            V[where] = rng.standard_normal((hk, 128))
            value = back(bits(V[where])).astype(np.float64)
        dp.write(f.node_pages[f.page_begin[v]: f.page_begin[v] + f.n_pages[v]], 0, gpu.to_device_bits(bits(K)), gpu.to_device_bits(bits(V)))
    q = np.zeros((n_req * T, hq, 128), dtype=np.float32)
    q[:, :, 0] = rng.uniform(0.3, 7.7, (n_req * T, hq))
    q[:, :, 1] = 1.0
    q = bits(q)
    masks = np.tile(np.asarray([(1 << (t + 1)) - 1 for t in range(T)], dtype=np.uint64), n_req) if T > 16 else None
    plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, hq, tokens_per_req=T, visible=masks, **settings)
    assert (hkv.hkv_decode_plan_num_tile_items(plan) > 0) == tiles
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    out = torch.zeros((n_req * T, hq, 128), dtype=torch.int16, device="cuda")
    hkv.attn_decode_plan_run(plan, gpu.to_device_bits(q), float(np.log(2.0)), out, None, torch.empty(nb, dtype=torch.uint8, device="cuda"), nb)
    torch.cuda.synchronize()
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()
    got, value = gpu.bf16_tensor_to_f64(out), np.repeat(value, hq // hk, axis=0)
    factor = (got * value).sum(axis=2) / (value * value).sum(axis=1)
    p = np.exp2(back(q)[:, :, 0].astype(np.float64))
    return factor / (p / (2.0 + p)) - 1.0


# With the row's maximum as reference that weight is exp2(0) = 1, exact in bf16, and what is left is the rounding of the 128 results:
# 2^-8 / sqrt(3) * 0.72 = 1.6e-3 rms each (0.72: mean place in a binade), times sqrt(sum v^4) / sum v^2 = sqrt(3 / 128): 2.5e-4.  With
# another reference the weight itself is rounded, 1.6e-3 rms.  The line between them is their geometric mean.
WEIGHT_RMS = 6.4e-4


@pytest.mark.parametrize("flags", [WIDE, NARROW])
@pytest.mark.parametrize("n_req, where", [(5, 69), (8, 145), (16, 256 + 31), (16, 500), (13, 64), (16, 96)])
def test_heaviest_weight_is_exact(gpu, flags, n_req, where):  # noqa: F811
    err = weight_of_one_key(gpu, n_req, 1, 640, where, flags=flags)
    assert np.sqrt((err ** 2).mean()) < WEIGHT_RMS


def test_heaviest_weight_of_drafted_rows_is_exact(gpu):  # noqa: F811
    """64 requests x 21 drafted tokens over 2048 shared tokens: 45 GFLOP above the last nodes, not on the one-reference tile."""
    err = weight_of_one_key(gpu, 64, 21, 2048, 1500, hq=32, hk=8)
    assert np.sqrt((err ** 2).mean()) < WEIGHT_RMS


@pytest.mark.parametrize("T, flags, settings, forks", [
    (1, 0, {"tile_min_gflop": -1, "fused": -1}, True), (1, 4, {"tile_min_gflop": -1, "fused": -1}, False),   # HKV_PLAN_ONE_STREAM
    (1, 0, {"tile_min_gflop": -1}, False),                                                              # one launch
    (8, 0, {"tile_min_gflop": 1}, False)])                                                               # tiles in front of the rest
def test_a_plan_holds_a_stream_only_if_its_runs_fork(gpu, T, flags, settings, forks):  # noqa: F811
    from paper_2603_16104_amd import binding as hkv
    n_req = 48 if T == 8 else 80
    parent, ntok = [-1] + [0] * n_req, [1040] + [T + 20] * n_req
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(1, n_req + 1)), np.arange(n_used, dtype=np.int32))
    dp = gpu.DevicePool(n_used, 2, wl.KV_FP8_E4M3)
    plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, 8, flags, tokens_per_req=T, **settings)
    assert hkv.hkv_decode_plan_num_tile_items(plan) > 0
    assert hkv.hkv_decode_plan_is_fused(plan) == ("fused" not in settings and T == 1)
    assert hkv.hkv_decode_plan_has_stream(plan) == forks
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()
