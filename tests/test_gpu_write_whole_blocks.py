"""kv_pool_write: blocks written whole next to blocks written in part, odd and even numbers of KV heads (a workgroup of an fp8 write of
400 blocks x heads or more takes two), and the numbers of blocks at which another size of kernel arguments, or none, is used: bytes
and scales equal the oracle's."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("H", [1, 2, 3, 8])
def test_whole_and_partial_blocks(gpu, oracle, kv_dtype, H):  # noqa: F811
    import torch
    least = -(-400 // H) * 16
    for first, tokens in [(0, least - 16), (0, least), (0, least + 1), (0, least + 15), (5, least - 5), (5, least), (5, least + 11), (5, least + 12), (15, least + 2),
                          (0, 960 * 16), (7, 960 * 16), (0, 1), (0, 15), (0, 16), (0, 17), (0, 32), (0, 47), (5, 3), (5, 11), (5, 12), (5, 27), (5, 28), (7, 50), (15, 1), (15, 33),
                          (0, 64 * 16), (0, 64 * 16 + 1), (3, 256 * 16 - 3), (3, 256 * 16 - 2)]:
        n_pages = (first + tokens + 15) // 16
        rng = np.random.default_rng([H, first, tokens])
        pages = rng.permutation(n_pages + 3)[:n_pages].astype(np.int32)
        hp, dp = oracle.HostPool(n_pages + 3, H, kv_dtype), gpu.DevicePool(n_pages + 3, H, kv_dtype)
        for slot, n in ([(0, first)] if first else []) + [(first, tokens)]:
            k, v = (wl.f32_to_bf16_bits(rng.standard_normal((n, H, 128)).astype(np.float32) * np.float32(1 + slot)) for _ in range(2))
            hp.write(pages, slot, k, v)
            dp.write(pages, slot, gpu.to_device_bits(k), gpu.to_device_bits(v))
        torch.cuda.synchronize()
        for name in ("k", "v") + (("k_scale", "v_scale") if kv_dtype == wl.KV_FP8_E4M3 else ()):
            got, exp = getattr(dp, name).cpu().numpy().view(np.uint8).ravel(), getattr(hp, name).view(np.uint8).ravel()
            if name.endswith("scale"):     # (unset scales: NaN of any kind)
                got, exp = (np.nan_to_num(x.view(np.float32), nan=-1.0) for x in (got, exp))
            assert np.array_equal(got, exp), (name, first, tokens)
        dp.close()
