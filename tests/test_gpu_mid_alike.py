"""Tensors of up to 64 K elements whose keys are alike, sorted or few: the list made a second time, its guess from a sample, and what that costs."""
import numpy as np
import pytest
import torch

import gpu_harness as H
from oracle import adatopk_oracle as orc
from paper_2410_12707_amd import binding as B
from paper_2410_12707_amd import workloads as wl

pytestmark = pytest.mark.gpu


def cast(x, dtype):
    return wl.f32_to_bf16_bits(x) if dtype == "bf16" else x.astype(np.float16) if dtype == "f16" else x.astype(np.float32)


def check(xs, ks):
    gi, gv, _, ge = H.gpu_compress_segmented(xs, ks)
    ri, rv, _, re = orc.compress_segmented(xs, ks)
    assert np.array_equal(gi, ri) and np.array_equal(H.bits(gv), H.bits(rv)), ks
    assert all(H.same_err(a, b) for a, b in zip(ge, re)), ks


def sampled(n):
    """Which elements the sample takes: one of sixteen consecutive ones in each group of 256."""
    i = np.arange(n)
    groups = -(-n // 256)
    first = np.arange(17) * groups // 16  # of each wavefront
    group = i // 256
    j = group - first[np.searchsorted(first, group, side="right") - 1]
    return (((i % 256) // 4) % 4 == j % 4) & (i % 4 == j // 4)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n", [16_385, 33_001, 51_200])
def test_a_sample_that_is_no_help(dtype, n):
    take, rng = sampled(n), np.random.default_rng(n)
    assert abs(take.mean() - 1 / 16) < 0.002
    for others in (np.full(n, 3.0), 3.0 + rng.integers(0, 2, n) * 0.25, 3.0 + rng.integers(0, 40, n) / 64):
        x = np.where(take, 1.0, others) * np.where(rng.random(n) < 0.5, -1, 1)
        a = np.sort(np.abs(x))[::-1]
        for k in (1, n // 200, n // 100):
            check([cast(x, dtype)], [k])
        for level in (3.25, 3.5):  # about where one key ends
            k = int((a >= level).sum())
            for k in (k - 1, k, k + 1):
                if 0 <= k <= n // 100:
                    check([cast(x, dtype)], [k])


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_keys_that_end_at_the_kept_number(dtype):
    for n in (9000, 16_384, 16_640, 36_000, 51_200):
        rng = np.random.default_rng(n)
        xs, ks = [], []
        for shares in ((0.004, 0.3), (0.01, 0.01, 0.5), (0.0005, 0.008, 0.9), (0.005, 0.0, 0.0)):
            x = np.zeros(n)
            order, at, value = rng.permutation(n), 0, 4.0
            for share in shares:
                count = int(n * share)
                x[order[at:at + count]] = value
                at, value = at + count, value - 0.5
                for k in (at - 1, at, at + 1):
                    if 0 <= k <= n // 100:
                        xs.append(cast(x, dtype))
                        ks.append(k)
        check(xs, ks)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n", [8193, 12_345, 16_384, 16_385, 20_000, 40_001, 51_200])
def test_alike_sorted_and_uneven(dtype, n):
    rng = np.random.default_rng(n)
    up = np.sort(np.abs(rng.standard_normal(n)))
    kinds = [up, up[::-1], np.sort(rng.standard_normal(n)), 1.0 + 0.03 * rng.random(n), 1.0 + 0.2 * rng.random(n), np.round(rng.standard_normal(n) * 32) / 32,
             np.round(rng.standard_normal(n) * 2) / 2, rng.standard_normal(n) * np.exp(np.repeat(rng.standard_normal(n // 1600 + 1), 1600)[:n]),
             np.full(n, -2.5), np.where(rng.random(n) < 0.995, 0.0, rng.standard_normal(n))]
    xs = [cast(x, dtype) for x in kinds]
    for k in (1, n // 300, n // 100, n // 100 + 1, n // 60):
        check(xs, [k] * len(xs))


def times(x, k, tensors):
    """The least time of every kernel of a call."""
    ks = [k] * tensors
    off = [k * i for i in range(tensors + 1)]
    idx, val = torch.empty(off[-1], dtype=torch.int32, device="cuda"), torch.empty(off[-1], dtype=x.dtype, device="cuda")
    ws, least = B.new_workspace(x.numel() * tensors, tensors, x.dtype), {}
    xs = [x.clone() for _ in range(tensors)]
    with B.measuring():
        for _ in range(8):
            B.adatopk_compress_segmented(xs, ks, idx, val, off, None, ws)
            torch.cuda.synchronize()
            for name, t in zip(B.measure_stage_names(), B.measure_read()):
                if t > 0:
                    least[name] = min(t, least.get(name, t))
    return least


@pytest.mark.parametrize("n,most", [(8192, 2.0), (65_536, 2.2)])
def test_alike_and_sorted_keys_cost_no_several_times_more(n, most):
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, device="cuda", generator=gen)
    usual = times(x, n // 100, 64)["k_mid"]
    for y in (1.0 + 0.03 * torch.rand(n, device="cuda", generator=gen), x.abs().sort().values, torch.ones_like(x)):
        assert times(y, n // 100, 64)["k_mid"] < most * usual


@pytest.mark.parametrize("dtype,n,share,kernel", [
    ("f32", 65_536, 0.01, "k_mid"), ("f32", 60_000, 0.05, "k_scan"),  # n + 13 k about 83 K
    ("bf16", 32_768, 0.03, "k_mid"), ("bf16", 50_000, 0.01, "k_scan"),  # ... 52 K
    ("f32", 8192, 0.2, "k_mid"), ("f32", 7000, 0.1, "k_small"), ("f32", 6000, 0.01, "k_mid"), ("f32", 4096, 0.01, "k_small")])
def test_calls_that_would_lose_take_the_other_kernels(dtype, n, share, kernel):
    x = torch.randn(n, device="cuda").to({"f32": torch.float32, "bf16": torch.bfloat16}[dtype])
    assert kernel in times(x, int(n * share), 24)
