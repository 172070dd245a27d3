"""Batches with tensors that keep so much that their chunks have no lists and are placed from the input: the results against the
oracle, as pairs and as wire messages, and into how many parts the chunks were cut."""
import struct

import numpy as np
import pytest

from oracle import adatopk_oracle as orc
from oracle import wire_format as wf
from paper_2410_12707_amd import workloads as wl
from test_gpu_parity import ERR_RTOL, check_segmented_decompress

pytestmark = pytest.mark.gpu


def compress(xs, ks):
    """Pairs, offsets, error norms and how many parts of chunks k_refine had something to do for (fp32)."""
    import torch

    import gpu_harness as H
    from paper_2410_12707_amd import binding as B

    ds = [H.to_device(x) for x in xs]
    off = [0]
    for k in ks:
        off.append(off[-1] + k)
    idx = torch.full((off[-1],), -7, dtype=torch.int32, device="cuda")
    val = torch.zeros(off[-1], dtype=ds[0].dtype, device="cuda")
    err = torch.full((len(xs),), -1.0, device="cuda")
    n_total = sum(x.size for x in xs)
    ws = B.new_workspace(n_total, len(xs), ds[0].dtype)
    ws.fill_(255)
    B.adatopk_compress_segmented(ds, ks, idx, val, off, err, ws)
    torch.cuda.synchronize()
    at = B.measure_workspace_offset(B.MEASURE_PART_COUNTS, n_total, len(xs), ds[0].dtype)
    room = 8 * 512 if len(xs) > 1 else 4 * 256  # most parts per chunk, most chunks
    parts = int((ws[at:at + 4 * room].view(torch.int32) != -1).sum()) if ds[0].dtype == torch.float32 else 0
    return H.to_host(idx), H.to_host(val), off, H.to_host(err), parts


def check(xs, ks):
    import gpu_harness as H

    gi, gv, off, ge, parts = compress(xs, ks)
    refs = [orc.compress(x, k) for x, k in zip(xs, ks)]
    for s, (ri, rv, re) in enumerate(refs):
        assert np.array_equal(gi[off[s]:off[s + 1]], ri) and np.array_equal(H.bits(gv[off[s]:off[s + 1]]), H.bits(rv)), s
        assert H.same_err(ge[s], re, ERR_RTOL), (s, ge[s], re)
    check_segmented_decompress(gi, gv, off, [x.size for x in xs])
    return parts, refs


def test_dense_tensors_beside_sparse_ones_are_cut_into_parts():
    # too few elements of either kind for launches of their own: the dense tensors' chunks go through the entry loop of the plain
    # kernels, with several workgroups to a chunk
    lens, shares = [8_400_003, 6_000_001, 3_000_000], [0.01, 0.6, 0.9]
    xs = [wl.small_case("normal", n, seed=200 + i) for i, n in enumerate(lens)]
    assert check(xs, [int(n * f) for n, f in zip(lens, shares)])[0] > 512


@pytest.mark.parametrize("dtype,tensors,n,keep", [("f32", 8, 1 << 20, 0.7), ("f32", 1, 4 << 20, 0.8), ("f32", 2, (14 << 20) - 8, 0.6),
                                                  ("f32", 2, 14 << 20, 0.6), ("f32", 1, (5 << 20) - 1, 0.9), ("f32", 1, 5 << 20, 0.9),
                                                  ("bf16", 1, 13 << 20, 0.3), ("bf16", 2, 13 << 19, 0.3), ("f16", 2, (13 << 19) - 4, 0.5)])
def test_one_part_per_chunk_only_from_a_total_length_on(dtype, tensors, n, keep):
    # either side of the lines between the list kernels' two forms; one workgroup per chunk where the wide one runs, several below
    xs = [wl.small_case("normal", n, seed=230 + i, dtype=dtype) for i in range(tensors)]
    written = check(xs, [int(n * keep)] * tensors)[0]
    chunks = 512 if tensors > 1 else 256
    if dtype == "f32":
        assert (written <= chunks) == (n * tensors >= (28 if tensors > 1 else 5) << 20), written


@pytest.mark.parametrize("tensors,n,keep,tiles,parts", [(2, 10 << 20, 0.7, 5, 4), (8, 3 << 19, 0.55, 3, 2), (4, 2 << 20, 0.9, 2, 2)])
def test_parts_of_chunks_without_lists_have_a_tile_each(tensors, n, keep, tiles, parts):
    # (with eight parts to chunks of five tiles, and four to chunks of three or two, the last ones have nothing to do or half a tile)
    xs = [wl.small_case("normal", n, seed=220 + i) for i in range(tensors)]
    chunks = -(-n // (tiles * 8192))
    last = n - (chunks - 1) * tiles * 8192  # elements of the last chunk; parts are multiples of 2048 elements
    written = check(xs, [int(n * keep)] * tensors)[0]
    assert written <= tensors * chunks * parts and written >= tensors * ((chunks - 1) * parts + min(parts, -(-last // 8192))), written


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sparse,dense,held", [(9 << 20, 0, 1), (9 << 20, 4_000_003, 1), (9 << 20, 5_000_001, 0), (8 << 20, 70_001, 1),
                                               ((8 << 20) - 8, 70_001, 0)])
def test_a_batch_speculates_where_most_of_it_can(dtype, sparse, dense, held):
    import torch

    import gpu_harness as H
    from paper_2410_12707_amd import binding as B

    lens, shares = [sparse // 2, dense, sparse // 2], [0.01, 0.3, 0.02]
    xs = [wl.small_case("normal", n, seed=240 + i, dtype=dtype) for i, n in enumerate(lens)]
    ks = [int(n * f) for n, f in zip(lens, shares)]
    check(xs, ks)
    ds = [H.to_device(x) for x in xs]
    off = [0, ks[0], ks[0] + ks[1], sum(ks)]
    ws = B.new_workspace(sum(lens), 3, ds[0].dtype)
    B.adatopk_compress_segmented(ds, ks, torch.empty(off[3], dtype=torch.int32, device="cuda"),
                                 torch.empty(off[3], dtype=ds[0].dtype, device="cuda"), off, None, ws)
    torch.cuda.synchronize()
    state = ws[:192].view(torch.int32).cpu()  # a record of 64 bytes per tensor, its seventh word the verdict
    assert state[6] == held and state[32 + 6] == held


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_chunks_of_many_tiles_without_lists(dtype):
    # more than 256 chunks of five tiles and more, and no workgroups for the error norms alone; ragged, and with a sparse and an empty
    # tensor between them; as pairs and as wire messages
    import torch

    import gpu_harness as H
    from paper_2410_12707_amd import binding as B

    lens, shares = [9_000_011, 0, 11_000_003, 50_000, 10_000_001], [0.55, 0.0, 0.95, 0.02, 0.8]
    xs = [wl.small_case("normal", n, seed=210 + i, dtype=dtype) for i, n in enumerate(lens)]
    ks = [int(n * f) for n, f in zip(lens, shares)]
    refs = check(xs, ks)[1]
    ds = [H.to_device(x) for x in xs]
    at, pos = [], 0
    for k in ks:
        at.append(pos)
        pos += (wf.message_bytes(k, xs[0].dtype, 4) + 15) // 16 * 16
    wire = torch.zeros(pos, dtype=torch.uint8, device="cuda")
    B.adatopk_compress_wire_segmented(ds, ks, 4, None, wire, at, B.new_workspace(sum(lens), len(lens), ds[0].dtype))
    torch.cuda.synchronize()
    raw = wire.cpu().numpy().tobytes()
    for s, (k, (ri, rv, re)) in enumerate(zip(ks, refs)):
        ref = wf.pack(ri, rv, lens[s], float(re), lens[s] / k if k else 0.0, 4)
        got = raw[at[s]:at[s] + len(ref)]
        assert got[:12] == ref[:12] and got[16:] == ref[16:], s
        assert H.same_err(struct.unpack("<f", got[12:16])[0], re, ERR_RTOL), s
