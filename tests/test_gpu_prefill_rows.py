"""Prefill tiles whose rows fill one to all eight of a workgroup's wavefronts (those without rows only move K and V), and small batches
whose tiles run in pieces of a half or a quarter of the rows: the edges of wavefronts and pieces, key ranges on both sides of a
refill of the page-id window, sequences that end inside a block, against the oracle."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import LSE_ABS_FP8_PREFILL, both_pools, check_close, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq, hk, prefix, new, pieces", [
    (4, 1, 16, (8,), 0), (4, 1, 960, (9,), 0), (4, 1, 976, (16,), 0), (4, 1, 48, (17, 1), 0), (4, 1, 1088, (40, 33, 31), 8),   # 32-row edges
    (32, 8, 512, (128, 100, 97, 5), 184), (32, 8, 256, (64,), 32), (8, 2, 0, (65,), 6), (8, 2, 1024, (33,) * 3, 18), (5, 1, 240, (51, 52, 13), 12),
    (16, 1, 512, (16, 3), 5), (1, 1, 512, (256, 70), 6), (32, 8, 512, (32,) * 30, 0), (9, 3, 496, (29, 30), 12), (40, 8, 512, (128,) * 4, 192),
])
@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
def test_short_tiles_and_pieces(gpu, oracle, kv_dtype, hq, hk, prefix, new, pieces):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    parent, ntok = [-1] + [0] * len(new), [prefix] + list(new)
    n_pages = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(1, len(new) + 1)), np.random.default_rng([prefix, *new]).permutation(n_pages + 3).astype(np.int32))
    w = wl.Workload(name=f"{hq}_{hk}_{prefix}_{new}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=kv_dtype, num_pages=n_pages + 3, seed=prefix + len(new),
                    forest=f, mode="prefill", q_len=np.asarray(new, dtype=np.int32))
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    r = gpu.PrefillRunner(dp, w)
    assert hkv.hkv_prefill_plan_num_pieces(r.plan) == pieces
    for _ in range(2):
        r.out.fill_(0x7FC0)
        r.lse.fill_(float("nan"))
        r.run()
        torch.cuda.synchronize()
        check_close(gpu.bf16_tensor_to_f64(r.out), exp_o, w.name)
        check_lse(r.lse.cpu().numpy(), exp_l, w.name, tol=LSE_ABS_FP8_PREFILL if kv_dtype == wl.KV_FP8_E4M3 else 2e-3)
    r.close()
    dp.close()
