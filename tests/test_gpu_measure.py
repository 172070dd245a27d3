"""The measuring build's kernel times."""
import numpy as np
import pytest
import torch

from paper_2410_12707_amd import binding as B

pytestmark = pytest.mark.gpu


def test_launches_of_one_kernel_are_added_up():
    # ten tensors of which four keep more than a fifth: two groups of launches, and each by itself
    x = [torch.randn(8 << 20, device="cuda", generator=torch.Generator(device="cuda").manual_seed(i)) for i in range(10)]
    ks = [(8 << 20) // (2 if i < 4 else 100) for i in range(10)]

    def scan(which):
        xs, kk = [x[i] for i in which], [ks[i] for i in which]
        off = np.concatenate([[0], np.cumsum(kk)]).tolist()
        idx, val = torch.empty(off[-1], dtype=torch.int32, device="cuda"), torch.empty(off[-1], device="cuda")
        ws, times = B.new_workspace(sum(y.numel() for y in xs), len(xs), torch.float32), []
        with B.measuring():
            for _ in range(6):
                B.adatopk_compress_segmented(xs, kk, idx, val, off, None, ws)
                torch.cuda.synchronize()
                times.append(B.measure_read()[B.measure_stage_names().index("k_scan_spec")])
        return min(times)

    both, dense, listed = scan(range(10)), scan(range(4)), scan(range(4, 10))
    assert 0.85 * (dense + listed) < both < 1.15 * (dense + listed)
