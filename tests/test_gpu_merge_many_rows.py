"""The merge of 16384 rows and more: the edges of that number and of its 16 rows a workgroup, rows of one to eight partials side by side, and rows
without any.  Against the oracle."""
import numpy as np
import pytest

from paper_2603_16104_amd import binding as hkv, workloads as wl

from test_gpu_parity import both_pools, check_close, check_lse, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth", [1, 2, 3, 5, 7])
@pytest.mark.parametrize("hq, hk, n_req, dtype", [(8, 2, 2048, wl.KV_BF16), (8, 2, 2050, wl.KV_FP8_E4M3), (5, 1, 3277, wl.KV_BF16), (8, 1, 2047, wl.KV_BF16)])
def test_many_rows(gpu, oracle, depth, hq, hk, n_req, dtype):  # noqa: F811
    import torch
    # a chain of shared nodes; the requests' own leaves hang from all of its nodes, and some requests end at a shared node or have no token at all
    parent, ntok = list(range(-1, depth - 1)), [32] * depth
    leaves = []
    for r in range(n_req):
        if r % 97 == 5:
            parent.append(-1)
            ntok.append(0)
        elif r % 13 == 3:
            leaves.append(r % depth)
            continue
        else:
            parent.append(r % depth)
            ntok.append(1 + r % 16)
        leaves.append(len(parent) - 1)
    n_used = sum((t + 15) // 16 for t in ntok)
    f = wl.make_forest(parent, ntok, leaves, np.random.default_rng(depth).permutation(n_used + 3).astype(np.int32))
    w = wl.Workload(name=f"merge_{hq}_{hk}_{n_req}_{depth}", num_q_heads=hq, num_kv_heads=hk, kv_dtype=dtype, num_pages=n_used + 3, seed=9, forest=f,
                    mode="decode")
    hp, dp = both_pools(gpu, oracle, w)
    exp_o, exp_l = oracle.run_workload(w, hp)
    # odd depths: row i of the plan reads and writes row to[i]
    to = np.random.default_rng(1).permutation(n_req).astype(np.int32) if depth % 2 else None
    plan = hkv.hkv_decode_plan_create_ex(dp.handle, f.nodes, f.node_pages, f.req_leaf, hq, q_rows=to)
    at = np.arange(n_req) if to is None else to
    counts = hkv.hkv_decode_plan_part_counts(plan, n_req)
    assert counts.max() == depth + 1 and counts.min() == 0
    nb = hkv.hkv_decode_plan_workspace_bytes(plan)
    ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device="cuda")  # (what no item writes is NaN)
    q = np.empty_like(w.q())
    q[at] = w.q()
    out = torch.full((n_req, hq, 128), -1, dtype=torch.int16, device="cuda")
    lse = torch.full((n_req, hq), float("nan"), dtype=torch.float32, device="cuda")
    hkv.attn_decode_plan_run(plan, gpu.to_device_bits(q), float(w.scale), out, lse, ws, nb)
    torch.cuda.synchronize()
    hkv.hkv_decode_plan_destroy(plan)
    dp.close()
    check_close(gpu.bf16_tensor_to_f64(out)[at], exp_o, w.name)
    check_lse(lse.cpu().numpy()[at], exp_l, w.name)
