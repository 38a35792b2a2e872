"""The full-precision kernel with four heads to a workgroup: head ratios that four does and does not divide, the edges of its steps, rows
of very different lengths in one batch.  Against the oracle at the bound asked of fp32 inputs."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import both_pools, check_close_fp32, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def batch(gpu, oracle, hq, hk, lens):  # noqa: F811
    parent, ntok = [-1] * len(lens), list(lens)
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, list(range(len(lens))), np.random.default_rng(len(lens)).permutation(n_used + 3).astype(np.int32))
    w = wl.Workload(name=f"fp32_{hq}_{hk}_{max(lens)}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=wl.KV_FP32, num_pages=n_used + 3, seed=7,
                    forest=f, mode="decode", src_dtype="fp32")
    hp, dp = both_pools(gpu, oracle, w)
    return w, dp, *oracle.run_workload(w, hp)


@pytest.mark.parametrize("hq, hk", [(2, 1), (3, 1), (4, 1), (5, 1), (8, 2), (16, 1), (7, 1)])
@pytest.mark.parametrize("lens", [(140,) * 300, (129, 0, 1, 143, 144, 145, 700, 16) * 35, (140, 129) * 300, (100, 1, 128, 65) * 160])
def test_four_heads(gpu, oracle, hq, hk, lens):  # noqa: F811
    import torch
    w, dp, exp_o, exp_l = batch(gpu, oracle, hq, hk, lens)
    r = gpu.DecodeRunner(dp, w)
    for _ in range(2):
        r.out.fill_(float("nan"))
        r.lse.fill_(float("nan"))
        r.run()
        torch.cuda.synchronize()
        check_close_fp32(gpu.bf16_tensor_to_f64(r.out), exp_o, w.name)
        check_lse(r.lse.cpu().numpy(), exp_l, w.name, tol=1e-4)
    r.close()
    dp.close()
