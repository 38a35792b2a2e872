"""The full-precision kernel at the edges of its pages, of its 32-key steps and of the number of wavefronts a launch takes, for
head ratios with and without a last odd head, against the oracle at the bound asked of fp32 inputs."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import both_pools, check_close_fp32, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq, hk", [(2, 2), (6, 2), (8, 2), (5, 1), (16, 1)])
@pytest.mark.parametrize("lens", [(1, 15, 16, 17, 31, 32, 33, 64, 127, 0), (128, 129, 200, 255, 256, 3), (257, 288, 300, 511, 513, 900, 1)])
def test_fp32_rows_edges(gpu, oracle, hq, hk, lens):  # noqa: F811
    import torch
    parent, ntok = [-1] * len(lens), list(lens)
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(len(lens))), np.random.default_rng(len(lens)).permutation(n_used + 3).astype(np.int32))
    for mode in ("decode", "prefill"):
        w = wl.Workload(name=f"fp32_{mode}_{hq}_{hk}_{max(lens)}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=wl.KV_FP32, num_pages=n_used + 3, seed=7,
                        forest=f, mode=mode, src_dtype="fp32", q_len=np.minimum(np.asarray(lens, dtype=np.int32), 5) if mode == "prefill" else None)
        hp, dp = both_pools(gpu, oracle, w)
        exp_o, exp_l = oracle.run_workload(w, hp)
        r = (gpu.DecodeRunner if mode == "decode" else gpu.PrefillRunner)(dp, w)
        r.out.fill_(float("nan"))
        r.run()
        torch.cuda.synchronize()
        check_close_fp32(gpu.bf16_tensor_to_f64(r.out), exp_o, w.name)
        check_lse(r.lse.cpu().numpy(), exp_l, w.name, tol=1e-4)
        r.close()
        dp.close()


def one_row(gpu, K, V, q, q_heads, decode=True):  # noqa: F811
    """out, lse of one request's newest token over K / V [tokens][kv_heads][128], fp32, through a decode or a prefill plan."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    n, H = K.shape[0], K.shape[1]
    dp = gpu.DevicePool((n + 15) // 16, H, wl.KV_FP32)
    pages = np.arange((n + 15) // 16, dtype=np.int32)
    dp.write(pages, 0, torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    out = torch.full((1, q_heads, 128), 7.0, dtype=torch.float32, device="cuda")
    lse = torch.full((1, q_heads), 7.0, dtype=torch.float32, device="cuda")
    qd = torch.from_numpy(q).cuda()
    if decode:
        f = wl.make_forest([-1], [n], [0], pages)
        plan = hkv.hkv_decode_plan_create(dp.handle, f.nodes, f.node_pages, f.req_leaf, q_heads)
        hkv.attn_decode_plan_run(plan, qd, 1.0, out, lse, torch.empty(256, dtype=torch.uint8, device="cuda"), 256)
    else:
        plan = hkv.hkv_prefill_plan_create(dp.handle, np.asarray([0, 1]), pages[None], np.asarray([n]), q_heads)
        hkv.attn_prefill_plan_run(plan, qd, 1.0, out, lse)
    torch.cuda.synchronize()
    (hkv.hkv_decode_plan_destroy if decode else hkv.hkv_prefill_plan_destroy)(plan)
    dp.close()
    return out[0].cpu().numpy().astype(np.float64), lse[0].cpu().numpy().astype(np.float64)


def exact_row(K, V, q, q_heads, keep):
    """The same in float64 over the tokens `keep`."""
    o, ls = np.zeros((q_heads, 128)), np.zeros(q_heads)
    for h in range(q_heads):
        kvh = h // (q_heads // K.shape[1])
        s = K[keep, kvh].astype(np.float64) @ q[0, h].astype(np.float64)
        ls[h] = s.max() + np.log(np.exp(s - s.max()).sum())
        o[h] = np.exp(s - ls[h]) @ V[keep, kvh].astype(np.float64)
    return o, ls


def row_inputs(n, q_heads, kv_heads):
    rng = np.random.default_rng([n, q_heads])
    K = (0.1 * rng.standard_normal((n, kv_heads, 128))).astype(np.float32)
    V = rng.standard_normal((n, kv_heads, 128)).astype(np.float32)
    q = rng.standard_normal((1, q_heads, 128)).astype(np.float32)
    q[:, :, 0] = 1.0
    return K, V, q


@pytest.mark.parametrize("decode", [True, False])
@pytest.mark.parametrize("hq, hk", [(2, 2), (4, 2), (3, 1)])
@pytest.mark.parametrize("n, loud, where", [(30, 3, (7, 25)), (200, 60, (3, 61, 66, 199)), (700, 1, (0, 31, 32, 640)), (700, 690, (0, 40, 170, 300))])
def test_values_of_no_weight_take_no_part(gpu, decode, hq, hk, n, loud, where):  # noqa: F811
    """One key whose score passes the others by 500: their weights are zero in fp32, and infinities and NaN among their values
    (in the same 32-key step, in another step of the same wavefront behind or in front of it, in other wavefronts) do not show."""
    K, V, q = row_inputs(n, hq, hk)
    K[:, :, 0] = 0.0
    K[loud, :, 0] = 500.0
    keep = [t for t in range(n) if t not in where]
    exp_o, exp_l = exact_row(K, V, q, hq, keep)
    for i, t in enumerate(where):
        V[t, :, i::2] = (np.inf, -np.inf, np.nan)[i % 3]
    got_o, got_l = one_row(gpu, K, V, q, hq, decode)
    check_close_fp32(got_o, exp_o, "infinite values")
    check_lse(got_l, exp_l, "infinite values", tol=2e-3)   # a score of 500 in 32 additions: 32 * 500 * 2^-24 = 1e-3


@pytest.mark.parametrize("n, quiet", [(100, range(32, 64)), (600, range(32, 64)), (600, range(0, 32)), (600, range(96, 600))])
def test_keys_that_score_minus_infinity(gpu, n, quiet):  # noqa: F811
    """A wavefront's first keys, or all of its keys, score -inf: their weight is zero, the rest is plain attention."""
    K, V, q = row_inputs(n, 4, 2)
    K[list(quiet), :, 0] = -np.inf
    keep = [t for t in range(n) if t not in quiet]
    exp_o, exp_l = exact_row(K, V, q, 4, keep)
    got_o, got_l = one_row(gpu, K, V, q, 4)
    check_close_fp32(got_o, exp_o, "-inf scores")
    check_lse(got_l, exp_l, "-inf scores", tol=1e-4)


@pytest.mark.parametrize("value, tokens", [(np.nan, [5]), (np.nan, [150]), (np.nan, range(300)), (np.inf, [150]), (-np.inf, range(300))])
def test_scores_without_a_softmax_give_nan(gpu, value, tokens):  # noqa: F811
    """A NaN or +inf among a row's scores, or nothing but -inf: out is NaN and lse -inf, never a finite number."""
    K, V, q = row_inputs(300, 4, 2)
    K[list(tokens), 0, 0] = value                       # of KV head 0 only
    got_o, got_l = one_row(gpu, K, V, q, 4)
    exp_o, exp_l = exact_row(K[:, 1:], V[:, 1:], q[:, 2:], 2, range(300))
    assert np.isnan(got_o[:2]).all() and np.isneginf(got_l[:2]).all()
    check_close_fp32(got_o[2:], exp_o, "the other head")
    check_lse(got_l[2:], exp_l, "the other head", tol=1e-4)


def test_fp32_launch_of_more_than_two_to_the_31_threads(gpu):  # noqa: F811
    """131 075 queries x 128 heads over one page: a launch takes 131 072 of them, the rest goes out as a second one."""
    import torch
    from paper_2603_16104_amd import binding as hkv
    n, H = (1 << 31) // (128 * 64 * 2) + 3, 128
    dp = gpu.DevicePool(1, H, wl.KV_FP32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    K, V = (torch.randn((16, H, 128), device="cuda", generator=gen) for _ in range(2))
    dp.write(np.zeros(1, dtype=np.int32), 0, K, V)
    q = torch.randn((n, H, 128), device="cuda", generator=gen)
    out, lse = torch.full_like(q, float("nan")), torch.full((n, H), float("nan"), device="cuda")
    f = wl.make_forest([-1], [16], [0] * n, np.zeros(1, dtype=np.int32))
    plan = hkv.hkv_decode_plan_create(dp.handle, f.nodes, f.node_pages, f.req_leaf, H)
    hkv.attn_decode_plan_run(plan, q, 0.1, out, lse, torch.empty(256, dtype=torch.uint8, device="cuda"), 256)
    torch.cuda.synchronize()
    hkv.hkv_decode_plan_destroy(plan)
    assert not torch.isnan(lse).any() and not any(torch.isnan(out[a: a + 8192]).any() for a in range(0, n, 8192))
    rows = [0, 1, 70000, n - 5, n - 4, n - 3, n - 2, n - 1]
    s = (q[rows].double()[:, :, None, :] @ K.double().permute(1, 2, 0).contiguous()[None])[:, :, 0] * 0.1
    l = torch.logsumexp(s, dim=2)
    o = (torch.exp(s - l[:, :, None])[:, :, None, :] @ V.double().permute(1, 0, 2).contiguous()[None])[:, :, 0]
    check_close_fp32(out[rows].cpu().numpy().astype(np.float64), o.cpu().numpy(), "rows on both sides of the cut")
    check_lse(lse[rows].cpu().numpy(), l.cpu().numpy(), "rows on both sides of the cut", tol=1e-4)
    dp.close()
