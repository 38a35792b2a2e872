"""The full-precision kernel with the keys of few rows cut into shares: the edges of shares and steps, rows
of very different lengths in one batch, values that must not spread (infinities of weight zero, NaN), and what a caller without (enough)
workspace gets.  Against the oracle at the bound asked of fp32 inputs."""
import numpy as np
import pytest

from paper_2603_16104_amd import binding as hkv, workloads as wl

from test_gpu_fp32_rows import exact_row, row_inputs
from test_gpu_fp32_rows_heads import batch
from test_gpu_parity import both_pools, check_close_fp32, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


# whole (63 pages), then a share for every 8 pages of the longest row: 8, 9, 16 and 32 of them
@pytest.mark.parametrize("hq, hk", [(1, 1), (2, 1), (3, 1), (4, 1), (5, 1), (8, 2), (16, 1), (7, 1)])
@pytest.mark.parametrize("lens", [(1008, 500), (1009, 16, 17), (1024, 1, 0, 1023, 128), (1152, 1151, 129), (2048, 2047, 2033, 100, 0), (4112, 3000)])
def test_shares(gpu, oracle, hq, hk, lens):  # noqa: F811
    import torch
    w, dp, exp_o, exp_l = batch(gpu, oracle, hq, hk, lens)
    r = gpu.DecodeRunner(dp, w)
    for _ in range(2):
        r.out.fill_(float("nan"))
        r.lse.fill_(float("nan"))
        r.run()
        torch.cuda.synchronize()
        assert (hkv.hkv_decode_plan_workspace_bytes(r.plan) > 0) == (max(lens) > 63 * 16)
        check_close_fp32(gpu.bf16_tensor_to_f64(r.out), exp_o, w.name)
        check_lse(r.lse.cpu().numpy(), exp_l, w.name, tol=1e-4)
    r.close()
    dp.close()


@pytest.mark.parametrize("hq, hk, root, lens, shares", [(32, 8, 1120, (17, 32, 1, 31) * 4, 2), (8, 8, 1136, (16, 1, 64, 15) * 4, 2),
                                                        (24, 8, 1200, (100, 1, 7, 0) * 3, 2), (32, 8, 1008, (1, 16) * 5, 3), (6, 2, 0, (1152, 1151, 17, 0) * 12, 2)])
def test_two_and_three_shares(gpu, oracle, hq, hk, root, lens, shares):  # noqa: F811
    import torch
    parent, ntok = [-1] + [0 if root else -1] * len(lens), [root] + list(lens)
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(1, len(lens) + 1)), np.random.default_rng(root).permutation(n_used + 3).astype(np.int32))
    w = wl.Workload(name=f"fp32_{hq}_{hk}_{root}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=wl.KV_FP32, num_pages=n_used + 3, seed=7,
                    forest=f, mode="decode", src_dtype="fp32")
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    r = gpu.DecodeRunner(dp, w)
    assert hkv.hkv_decode_plan_workspace_bytes(r.plan) == 528 * len(lens) * hq * shares
    r.out.fill_(float("nan"))
    r.lse.fill_(float("nan"))
    r.run()
    torch.cuda.synchronize()
    check_close_fp32(gpu.bf16_tensor_to_f64(r.out), exp_o, w.name)
    check_lse(r.lse.cpu().numpy(), exp_l, w.name, tol=1e-4)
    r.close()
    dp.close()


def test_workspaces(gpu, oracle):  # noqa: F811
    """None, too small, misaligned and the static form: whole rows; enough: shares.  All the same numbers but for the order of 32-bit sums."""
    import torch
    w, dp, exp_o, exp_l = batch(gpu, oracle, 8, 2, (2000, 1234, 77))
    f = w.forest
    plan = hkv.hkv_decode_plan_create(dp.handle, f.nodes, f.node_pages, f.req_leaf, 8)
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    assert nb > 0
    ws = torch.zeros(nb + 4096, dtype=torch.uint8, device="cuda")
    q = torch.from_numpy(w.q()).cuda()
    out, lse = (torch.empty(s, dtype=torch.float32, device="cuda") for s in ((3, 8, 128), (3, 8)))

    def check(run):
        out.fill_(float("nan"))
        ws.zero_()
        run()
        torch.cuda.synchronize()
        check_close_fp32(out.double().cpu().numpy(), exp_o, w.name)
        check_lse(lse.cpu().numpy(), exp_l, w.name, tol=1e-4)
        return bool(ws.any())

    scale = float(w.scale)
    assert check(lambda: hkv.attn_decode_plan_run(plan, q, scale, out, lse, ws, nb))
    assert check(lambda: hkv.attn_decode_plan_run(plan, q, scale, out, None, ws, nb) or lse.copy_(torch.from_numpy(exp_l.astype(np.float32))))
    for give in ((None, 0), (ws, nb - 1), (ws[8:], nb)):
        assert not check(lambda: hkv.attn_decode_plan_run(plan, q, scale, out, lse, *give))
    assert not check(lambda: hkv.attn_decode_plan_run_static(plan, q, scale, out, lse))
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()


@pytest.mark.parametrize("hq, hk", [(4, 1), (8, 2), (5, 1)])
@pytest.mark.parametrize("what", ["v_inf_of_no_weight", "nan_score", "inf_score", "all_minus_inf_in_a_share", "all_minus_inf"])
def test_values_that_must_not_spread(gpu, hq, hk, what):  # noqa: F811
    import torch
    n = 1500
    K, V, q = row_inputs(n, hq, hk)
    K[:, :, 0] = 0.0
    keep = np.arange(n)
    if what == "v_inf_of_no_weight":          # a key 1000 below the others: its weight underflows, its infinite value takes no part
        K[700, :, 0] = -1000.0
        V[700] = np.inf
        keep = keep[keep != 700]
    elif what in ("nan_score", "inf_score"):
        K[700, 0, 0] = np.nan if what == "nan_score" else np.inf
    else:
        quiet = slice(128, 400) if what == "all_minus_inf_in_a_share" else slice(None)
        K[quiet, :, 0] = -np.inf
        keep = np.delete(keep, quiet)
    dp = gpu.DevicePool((n + 15) // 16, hk, wl.KV_FP32)
    pages = np.arange((n + 15) // 16, dtype=np.int32)
    dp.write(pages, 0, torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    f = wl.make_forest([-1], [n], [0], pages)
    plan = hkv.hkv_decode_plan_create(dp.handle, f.nodes, f.node_pages, f.req_leaf, hq)
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    assert nb > 0
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    out, lse = (torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in ((1, hq, 128), (1, hq)))
    hkv.attn_decode_plan_run(plan, torch.from_numpy(q).cuda(), 1.0, out, lse, ws, nb)
    torch.cuda.synchronize()
    got, got_l = out[0].double().cpu().numpy(), lse[0].double().cpu().numpy()
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()
    G = hq // hk
    bad = slice(0, 0) if what in ("v_inf_of_no_weight", "all_minus_inf_in_a_share") else slice(0, G) if what in ("nan_score", "inf_score") else slice(0, hq)
    assert np.isnan(got[bad]).all() and np.isneginf(got_l[bad]).all()     # as whole rows do
    rest = np.ones(hq, dtype=bool)
    rest[bad] = False
    if rest.any():
        with np.errstate(invalid="ignore"):   # (the bad rows too)
            exp, exp_l = exact_row(K, V, q, hq, keep)
        check_close_fp32(got[rest], exp[rest], what)
        assert np.abs(got_l[rest] - exp_l[rest]).max() <= 1e-4
