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
