"""lse_merge_dense at the numbers of slots per row where another kernel or another unrolling takes over: any count up to that number,
rows without partials, empty partials and unused slots that hold NaN, both result types."""
import numpy as np
import pytest

from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_groups, rows_per_count", [(7, 3), (2051, 8)])     # 21 rows; 16408: four rows per half wavefront
@pytest.mark.parametrize("max_parts", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 130])
def test_merge(gpu, n_groups, rows_per_count, max_parts):  # noqa: F811
    import torch
    from paper_2603_16104_amd import binding as hkv
    if n_groups > 100 and max_parts > 33:
        n_groups = 20
    n = n_groups * rows_per_count
    g = torch.Generator(device="cuda")
    g.manual_seed(max_parts)
    o = torch.randn((n, max_parts, 128), device="cuda", generator=g)
    lse = 4 * torch.randn((n, max_parts), device="cuda", generator=g)
    cnt = torch.randint(0, max_parts + 1, (n_groups,), device="cuda", generator=g, dtype=torch.int32)
    cnt[0], cnt[1] = max_parts, 0
    used = torch.arange(max_parts, device="cuda")[None, :] < cnt.repeat_interleave(rows_per_count)[:, None]
    empty = torch.rand((n, max_parts), device="cuda", generator=g) < 0.2
    empty[2] = True                                                       # a row whose partials are all empty
    lse[empty] = -torch.inf
    lse[~used] = torch.nan
    w = torch.where(used & ~empty, lse.double(), -torch.inf)
    exp_l = torch.logsumexp(w, 1)
    p = torch.where(torch.isneginf(exp_l)[:, None], 0.0, torch.exp(w - exp_l[:, None]))
    exp_o = torch.bmm(p[:, None, :], o.double())[:, 0]
    o[empty | ~used] = torch.nan
    for dtype, tdt, tol in ((hkv.FP32, torch.float32, 3e-6), (hkv.BF16, torch.bfloat16, 2 ** -8)):   # exp2 of a product with log2 e; half a bf16 unit
        out = torch.full((n, 128), 7.0, dtype=tdt, device="cuda")
        got_l = torch.full((n,), 7.0, device="cuda")
        hkv.lse_merge_dense(o, lse, cnt, rows_per_count, max_parts, n, out, dtype, got_l)
        torch.cuda.synchronize()
        assert torch.equal(torch.isneginf(got_l), torch.isneginf(exp_l))
        fin = ~torch.isneginf(exp_l)
        assert (got_l[fin] - exp_l[fin]).abs().max() <= 1e-5
        assert (out[~fin] == 0).all()
        err = (out.double() - exp_o).abs()
        assert (err <= tol * (p[:, None, :] @ torch.nan_to_num(o.double()).abs())[:, 0] + (2 ** -9 * exp_o.abs() if dtype == hkv.BF16 else 0)).all(), float(err.max())
