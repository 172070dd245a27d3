"""Batches of tensors that keep more than a fifth, 28 Mi fp32 or 13 Mi 16-bit elements of them in a call: a window from the sample, lists of the window's
bins alone, and the placing from the input."""
import numpy as np
import pytest

import gpu_harness as H
from oracle import adatopk_oracle as orc
from paper_2410_12707_amd import workloads as wl

pytestmark = pytest.mark.gpu
KINDS = ["normal", "few_levels", "sparse", "all_equal", "all_zero", "nonfinite", "random_bits", "descending"]
LEAST = {"f32": 28 << 20, "bf16": 13 << 20, "f16": 13 << 20}


def dense_held(xs, ks):
    """Which of the tensors, in the order of the launch for the dense ones, had a window that held."""
    import torch

    from paper_2410_12707_amd import binding as B

    ds = [H.to_device(x) for x in xs]
    off = np.concatenate([[0], np.cumsum(ks)]).tolist()
    ws = B.new_workspace(sum(x.size for x in xs), len(xs), ds[0].dtype)
    B.adatopk_compress_segmented(ds, ks, torch.empty(off[-1], dtype=torch.int32, device="cuda"),
                                 torch.empty(off[-1], dtype=ds[0].dtype, device="cuda"), off, None, ws)
    torch.cuda.synchronize()
    return ws[:64 * len(xs)].view(torch.int32).cpu()[6::16]


def check(xs, ks):
    gi, gv, off, ge = H.gpu_compress_segmented(xs, ks)
    for s, (x, k) in enumerate(zip(xs, ks)):
        ri, rv, re = orc.compress(x, k)
        assert np.array_equal(gi[off[s]:off[s + 1]], ri) and np.array_equal(H.bits(gv[off[s]:off[s + 1]]), H.bits(rv)), s
        assert H.same_err(ge[s], re), (s, ge[s], re)


def cast(x, dtype):
    return wl.f32_to_bf16_bits(x) if dtype == "bf16" else x.astype(np.float16) if dtype == "f16" else x


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_keep_shares_and_values(dtype):
    # tiles' edges, odd lengths, shares at both ends, beside ones that keep little, one that is kept whole and short ones
    ns = [1_048_576, 2_097_152, 1_048_577, 1_500_001, 2_000_003, 1_048_583, 1_700_000, 1_600_007]
    shares = [0.22, 0.3, 0.5, 0.75, 0.91, 0.995]
    xs, fs = [], []
    while sum(x.size for x in xs) < LEAST[dtype]:
        i = len(xs)
        xs.append(wl.small_case(KINDS[(i + i // 8) % 8], ns[i % 8], seed=i, dtype=dtype))
        fs.append(shares[i % 6])
    for n, f in ((9000, 0.4), (40_001, 1.0), (1_200_000, 0.01), (0, 0.0)):
        xs.insert(3, wl.small_case("normal", n, seed=n, dtype=dtype) if n else xs[0][:0])
        fs.insert(3, f)
    check(xs, [int(x.size * f) for x, f in zip(xs, fs)])


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_windows_that_miss_and_lists_that_overflow(dtype):
    n = (LEAST[dtype] // 6 + 3) | 1
    rng = np.random.default_rng(3)
    xs = [wl.small_case("normal", n, seed=50 + i) for i in range(6)]
    xs[0] *= np.repeat(np.exp(rng.standard_normal(n // 256 + 1) * 2), 256)[:n].astype(np.float32)  # runs of one scale: the sample sees few of them
    xs[1][: n // 2] *= np.float32(1e-3)  # two populations, the k-th key between them
    xs[2] = (1.0 + 0.02 * rng.random(n)).astype(np.float32)  # everything within the window: no lists
    xs[3] = np.round(xs[3] * 4).astype(np.float32) / 4
    xs = [cast(x, dtype) for x in xs]
    for shares in ((0.25, 0.5, 0.3, 0.5, 0.3, 0.6), (0.8, 0.499, 0.7, 0.8, 0.45, 0.95)):
        check(xs, [int(n * f) for f in shares])


def test_windows_hold_for_independent_values():
    n = 15 << 20
    xs = [wl.small_case("normal", n, seed=i) for i in range(2)]
    for shares in ((0.22, 0.35), (0.5, 0.7), (0.9, 0.8)):
        assert dense_held(xs, [int(n * f) for f in shares]).tolist() == [1, 1]
