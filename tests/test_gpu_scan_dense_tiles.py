"""Tiles of which more than a quarter are candidates, in launches of many chunks: lists stored group by group, and what sorted and equal values cost."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("length,share", [(900_001, 0.11), (900_001, 0.2), (4_500_003, 0.1)])  # exact passes; a list that overflows; from a sample
def test_blocks_of_candidates(dtype, length, share):
    xs, ks = [], []
    for t in range(3):
        rng = np.random.default_rng(t)
        x = rng.standard_normal(length) * 0.1
        for at in range(0, length, 32_768):  # whole groups, at any place in the list
            block = x[at + rng.integers(0, 9):][: int(32_768 * share) + rng.integers(0, 300)]
            block[:] = [np.sort(2 + rng.random(block.size))[::-1], np.full(block.size, -2.5), 2 + rng.random(block.size)][(t + at // 32_768) % 3]
        xs.append(cast(x, dtype))
        ks.append(int(length * share))
    gi, gv, off, ge = H.gpu_compress_segmented(xs, ks)
    for s, (x, k) in enumerate(zip(xs, ks)):
        ri, rv, re = orc.compress(x, k)
        assert np.array_equal(gi[off[s]:off[s + 1]], ri) and np.array_equal(H.bits(gv[off[s]:off[s + 1]]), H.bits(rv)), s
        assert H.same_err(ge[s], re), (s, ge[s], re)


def scan_time(xs, share):
    ks = [int(x.numel() * share) for x in xs]
    off = np.concatenate([[0], np.cumsum(ks)]).tolist()
    idx, val = torch.empty(off[-1], dtype=torch.int32, device="cuda"), torch.empty(off[-1], dtype=xs[0].dtype, device="cuda")
    ws, times = B.new_workspace(sum(x.numel() for x in xs), len(xs), xs[0].dtype), []
    with B.measuring():
        for _ in range(10):
            B.adatopk_compress_segmented(xs, ks, idx, val, off, None, ws)
            torch.cuda.synchronize()
            stages = dict(zip(B.measure_stage_names(), B.measure_read()))
            times.append(stages["k_scan_spec"] if stages["k_scan_spec"] > 0 else stages["k_scan"])
    return min(times)


def test_sorted_and_equal_values_cost_no_more_to_scan():
    x = [torch.randn(4_000_000, device="cuda", generator=torch.Generator(device="cuda").manual_seed(i)) for i in range(6)]
    assert scan_time([y.sort().values for y in x], 0.25) < 1.2 * scan_time(x, 0.25)
    one = x[0][:393_216]
    assert scan_time([torch.ones_like(one)], 0.01) < 1.2 * scan_time([one], 0.01)
