"""kv_pool_write around the number of blocks whose ids travel in the kernel's arguments (960): bytes and scales equal the
oracle's on both sides of that line, for calls that begin and end inside a block, and for pages of several blocks."""
import numpy as np
import pytest

from paper_2603_16104_amd import workloads as wl

from test_gpu_parity import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype", [wl.KV_BF16, wl.KV_FP8_E4M3])
@pytest.mark.parametrize("page_size, first, tokens", [
    (16, 0, 1), (16, 15, 2), (16, 0, 960 * 16), (16, 3, 960 * 16 - 3), (16, 3, 960 * 16 - 2), (16, 0, 961 * 16),
    (64, 37, 960 * 16 - 5), (64, 0, 240 * 64), (64, 0, 240 * 64 + 1)])
def test_write_at_the_inline_limit(gpu, oracle, kv_dtype, page_size, first, tokens):  # noqa: F811
    import torch
    H = 2
    rng = np.random.default_rng([page_size, first, tokens])
    n_pages = (first + tokens + page_size - 1) // page_size
    pages = rng.permutation(n_pages + 3)[:n_pages].astype(np.int32)
    hp = oracle.HostPool(n_pages + 3, H, kv_dtype, page_size=page_size)
    dp = gpu.DevicePool(n_pages + 3, H, kv_dtype, page_size=page_size)

    def write(slot, n):
        k = wl.f32_to_bf16_bits(rng.standard_normal((n, H, 128)).astype(np.float32))
        v = wl.f32_to_bf16_bits(rng.standard_normal((n, H, 128)).astype(np.float32))
        hp.write(pages, slot, k, v)
        dp.write(pages, slot, gpu.to_device_bits(k), gpu.to_device_bits(v))

    if first:
        write(0, first)        # the slots in front of a continued block have been written before
    write(first, tokens)
    torch.cuda.synchronize()
    for name in ("k", "v") + (("k_scale", "v_scale") if kv_dtype == wl.KV_FP8_E4M3 else ()):
        got, exp = getattr(dp, name).cpu().numpy().view(np.uint8).ravel(), getattr(hp, name).view(np.uint8).ravel()
        if name in ("k", "v"):
            assert np.array_equal(got, exp), name
        else:                  # scales of blocks that were never written differ in their poison only
            g, e = got.view(np.float32), exp.view(np.float32)
            assert np.array_equal(g[~np.isnan(e)], e[~np.isnan(e)]) and np.array_equal(np.isnan(g), np.isnan(e)), name
    dp.close()


def test_codes_at_ties_and_extreme_scales(gpu, oracle):  # noqa: F811
    """fp8 codes where the quotient x / scale lies on or next to the middle between two codes, for zeros of both signs, and in
    blocks whose scale is tiny, huge or subnormal (those divide; the others go by the reciprocal): bytes equal the oracle's."""
    import torch
    rng = np.random.default_rng(3)
    H, n_blk = 2, 64
    x = np.zeros((n_blk * 16, H, 128), dtype=np.float32)
    for b in range(n_blk):
        amax = np.float32(1.0 + rng.integers(0, 128) / 128.0) * np.float32(2.0) ** [0, 0, 0, 3, -7, 60, -50, -51, -52, 68, 69, 70, -118, -125, 100, -100][b % 16]
        mid = rng.choice(np.asarray([0, 1, 3, 5, 7, 9, 11, 13, 15, 17, 21, 25, 30, 104, 120, 232, 248, 416, 432], dtype=np.float32), (16, H, 128))
        v = np.float32(amax) * mid / np.float32(448.0) * rng.choice(np.asarray([1, -1, 0.5, 2 ** -9, 2 ** -10], dtype=np.float32), (16, H, 128))
        v[0, :, 0] = amax
        v[1, :, 1] = -0.0
        x[16 * b: 16 * b + 16] = np.clip(v, -amax, amax)
    k = wl.f32_to_bf16_bits(x)
    v = wl.f32_to_bf16_bits(np.ascontiguousarray(x[:, :, ::-1]))
    pages = rng.permutation(n_blk).astype(np.int32)
    hp, dp = oracle.HostPool(n_blk, H, wl.KV_FP8_E4M3), gpu.DevicePool(n_blk, H, wl.KV_FP8_E4M3)
    hp.write(pages, 0, k, v)
    dp.write(pages, 0, gpu.to_device_bits(k), gpu.to_device_bits(v))
    torch.cuda.synchronize()
    for name in ("k", "v", "k_scale", "v_scale"):
        assert np.array_equal(getattr(dp, name).cpu().numpy().view(np.uint8).ravel(), getattr(hp, name).view(np.uint8).ravel()), name
    dp.close()
