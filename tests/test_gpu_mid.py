"""Tensors of up to 64 K elements, selected in one launch by one workgroup each: its groups of 256 elements, its three ways to bound the k-th
key, its list and the way without one."""
import numpy as np
import pytest

import gpu_harness as H
from oracle import adatopk_oracle as orc
from paper_2410_12707_amd import workloads as wl

pytestmark = pytest.mark.gpu
KINDS = ["normal", "near_one", "blocks", "few_levels", "sparse", "all_equal", "all_zero", "nonfinite", "random_bits", "descending"]


def values(kind, n, seed, dtype):
    if kind == "near_one":  # all keys within a bin of the bound's histogram
        x = (1.0 + 0.03 * np.random.default_rng(seed).random(n)).astype(np.float32)
    elif kind == "blocks":  # zeros but for one block
        x = wl.small_case("normal", n, seed=seed)
        x[: n // 3] = 0.0
        x[n // 3 + 700:] = 0.0
    else:
        return wl.small_case(kind, n, seed=seed, dtype=dtype)
    return wl.f32_to_bf16_bits(x) if dtype == "bf16" else x.astype(np.float16) if dtype == "f16" else x


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n", [8193, 8447, 12_289, 16_383, 16_385, 40_001, 65_281, 65_535, 65_536])
def test_every_keep_count(dtype, n):
    # the limits between one, four and sixteen maxima per thread (640, 2560), and those of the path (n + 13 k up to 2^17, n / 4), on both sides
    ks = [0, 1, 2, 639, 640, 641, 2560, 2561, n // 100, n // 7, n // 5, n // 4, n // 4 + 1, n // 2, n - 1, n, ((1 << 17) - n) // 13, ((1 << 17) - n) // 13 + 1]
    xs = [values(kind, n, n % 777 + i, dtype) for i, kind in enumerate(KINDS)]
    xs += [xs[0]] * (-(-(1 << 20) // n) - len(xs))  # (a call of 2^20 elements)
    for k in (k for k in ks if k <= n):
        gi, gv, off, ge = H.gpu_compress_segmented(xs, [k] * len(xs))
        ri, rv, roff, re = orc.compress_segmented(xs, [k] * len(xs))
        assert np.array_equal(gi, ri) and np.array_equal(H.bits(gv), H.bits(rv)), k
        for s, kind in enumerate(KINDS):
            assert H.same_err(ge[s], re[s]), (k, kind, ge[s], re[s])


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_more_tensors_than_one_launch_holds(dtype):
    rng = np.random.default_rng(7)
    lens = [0, 1, 63, 257, 9000, 65_536, 0] + rng.integers(1, 40_000, size=200).tolist()
    xs = [wl.small_case("normal", n, seed=i, dtype=dtype) if n else wl.small_case("normal", 1, 1, dtype)[:0] for i, n in enumerate(lens)]
    ks = [int(n * 0.02) for n in lens]
    gi, gv, _, ge = H.gpu_compress_segmented(xs, ks)
    ri, rv, _, re = orc.compress_segmented(xs, ks)
    assert np.array_equal(gi, ri) and np.array_equal(H.bits(gv), H.bits(rv))
    assert all(H.same_err(a, b) for a, b in zip(ge, re))


@pytest.mark.parametrize("longest", [4096, 4097, 4100, 5121, 8191, 8192])  # the last length of the other kernel, and this one's
def test_calls_of_small_tensors(longest):
    # beside tensors of which most wavefronts, or most lanes of the last one, have no element; the call uses no workspace
    lens = [longest, 0, 4, 5, 63, 64, 65, 255, 256, 257, 600, 1023, 4095, longest - 1]
    for kind in KINDS:
        xs = [values(kind, max(n, 1), longest + i, "f32")[:n] for i, n in enumerate(lens)]
        for share in (0.0, 0.003, 0.25):
            ks = [int(n * share) for n in lens]
            gi, gv, _, ge = H.gpu_compress_segmented(xs, ks)
            ri, rv, _, re = orc.compress_segmented(xs, ks)
            assert np.array_equal(gi, ri) and np.array_equal(H.bits(gv), H.bits(rv)), (kind, share)
            assert all(H.same_err(a, b) for a, b in zip(ge, re)), (kind, share)
