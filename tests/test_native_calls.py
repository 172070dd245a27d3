"""The calls that the _marshal extension makes: it leaves to Python whatever is not plain, and with it a call does and refuses the same."""
import numpy as np
import pytest
import torch

from paper_2410_12707_amd import binding as B


def test_what_is_not_plain_is_left_to_python():
    m, lib = B._load_marshal(), B.load_library()
    x, idx, val, ws = torch.zeros(64), torch.zeros(8, dtype=torch.int32), torch.zeros(8), torch.zeros(256, dtype=torch.uint8)  # not in device memory
    assert m.compress(lib.address.compress, x, 8, idx, val, None, ws) is None
    assert m.decompress(lib.address.decompress, idx, val, 8, x) is None
    assert m.decompress_wire(lib.address.decompress_wire, ws, 128, 4, x, False) is None
    assert m.compress_wire(lib.address.compress_wire, x, 8, 4, 8.0, ws, ws) is None
    assert m.compress_segmented(lib.address.compress_segmented, [x, x], [4, 4], idx, val, [0, 4, 8], None, ws) is None
    assert m.compress_segmented(lib.address.compress_segmented, [], [], idx, val, [0], None, ws) is None
    assert m.decompress_segmented(lib.address.decompress_segmented, idx, val, [0, 8], [x]) is None
    assert m.compress_wire_segmented(lib.address.compress_wire_segmented, [x], [8], 4, None, ws, [0], ws) is None
    for wrong in ((None,) * 7, ("x", 1, 2.0, [], {}, (), 0)):
        assert m.compress(*wrong) is None
    with pytest.raises(TypeError):
        m.compress(1, 2)
    with pytest.raises(ValueError):
        B.adatopk_compress(x, 8, idx, val, None, ws)


@pytest.mark.gpu
def test_calls_with_and_without_the_extension(monkeypatch):
    rng = np.random.default_rng(1)
    xs = [torch.from_numpy(rng.standard_normal(n).astype(np.float32)).cuda() for n in (5000, 300_000, 70_000)]
    ks = [50, 3000, 700]
    off = [0, 50, 3050, 3750]
    at = [0, 1024, 32_768]

    def everything():
        out = []
        idx, val, err = torch.zeros(off[3], dtype=torch.int32, device="cuda"), torch.zeros(off[3], device="cuda"), torch.zeros(3, device="cuda")
        ws = B.new_workspace(sum(x.numel() for x in xs), 3, torch.float32)
        ys = [torch.full_like(x, 7.0) for x in xs]
        wire = torch.zeros(65_536, dtype=torch.uint8, device="cuda")
        B.adatopk_compress_segmented(xs, ks, idx, val, off, err, ws)
        B.adatopk_decompress_segmented(idx, val, off, ys)
        out += [idx.clone(), val.clone(), err.clone()] + [y.clone() for y in ys]
        for call in (B.adatopk_decompress, B.adatopk_decompress_sorted, B.adatopk_decompress_accumulate):
            call(idx[50:3050], val[50:3050], 3000, ys[1])
            out.append(ys[1].clone())
        B.adatopk_compress(xs[1], ks[1], idx, val, None, ws)
        B.adatopk_compress_wire_segmented(xs, ks, 4, [100.0, 100.0, 100.0], wire, at, ws)
        for i in range(3):
            B.adatopk_decompress_wire(wire[at[i]:], B.adatopk_wire_bytes(ks[i], 0, 4), 4, ys[i], accumulate=i == 1)
        B.adatopk_compress_wire(xs[0], 50, 8, 100.0, wire, ws)
        torch.cuda.synchronize()
        return out + [idx, val, wire] + ys

    def refused():
        idx, val, ws = torch.zeros(100, dtype=torch.int32, device="cuda"), torch.zeros(100, device="cuda"), torch.zeros(256, dtype=torch.uint8, device="cuda")
        calls = [lambda: B.adatopk_compress(xs[1], 50, idx, val, None, ws),  # workspace
                 lambda: B.adatopk_compress(xs[1], 101, idx, val, None, ws),  # outputs
                 lambda: B.adatopk_compress(xs[1], -1, idx, val, None, ws),
                 lambda: B.adatopk_compress(xs[1][::2], 50, idx, val, None, ws),
                 lambda: B.adatopk_compress(xs[1].double(), 50, idx, val, None, ws),
                 lambda: B.adatopk_decompress(idx.long(), val, 50, xs[1]),
                 lambda: B.adatopk_decompress_wire(ws, 7, 4, xs[1]),
                 lambda: B.adatopk_decompress_wire(ws, 128, 5, xs[1]),
                 lambda: B.adatopk_compress_segmented([xs[0], xs[1].half()], [5, 5], idx, val, [0, 5, 10], None, ws),
                 lambda: B.adatopk_compress_segmented(xs, [5, 5], idx, val, [0, 5, 10, 15], None, ws),
                 lambda: B.adatopk_decompress_segmented(idx, val, [0, 5, 200], xs[:2])]
        kinds = []
        for call in calls:
            with pytest.raises(Exception) as e:
                call()
            kinds.append((e.type, str(e.value)))
        return kinds

    assert B._load_marshal()
    with_it, refused_with = everything(), refused()
    monkeypatch.setattr(B, "_marshal", False)
    without, refused_without = everything(), refused()
    assert all(torch.equal(a, b) for a, b in zip(with_it, without)) and refused_with == refused_without


@pytest.mark.gpu
def test_exceptions_of_python_code_end_the_call():
    m = B._load_marshal()
    x, idx, val, ws = torch.ones(64, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda"), torch.zeros(8, device="cuda"), B.new_workspace(64, 1, torch.float32)
    wire = torch.zeros(256, dtype=torch.uint8, device="cuda")
    calls = [lambda: B.adatopk_compress(x, 8, idx, val, None, ws), lambda: B.adatopk_decompress(idx, val, 8, x),
             lambda: B.adatopk_compress_wire(x, 8, 4, 8.0, wire, ws), lambda: B.adatopk_decompress_wire(wire, 128, 4, x),
             lambda: B.adatopk_compress_segmented([x], [8], idx, val, [0, 8], None, ws), lambda: B.adatopk_decompress_segmented(idx, val, [0, 8], [x]),
             lambda: B.adatopk_compress_wire_segmented([x], [8], 4, None, wire, [0], ws)]

    def interrupted(*_):  # as a signal's handler does while the stream is asked for
        raise KeyboardInterrupt

    for ways in ((interrupted, B._raw_stream), (torch.cuda.current_device, interrupted)):
        m.streams(*ways)
        try:
            for call in calls:
                with pytest.raises(KeyboardInterrupt):
                    call()
        finally:
            m.streams(torch.cuda.current_device, B._raw_stream)

    class Neither:
        def __bool__(self):
            raise ZeroDivisionError

    with pytest.raises(ZeroDivisionError):
        B.adatopk_decompress_wire(wire, 128, 4, x, accumulate=Neither())
    torch.cuda.synchronize()
    assert not idx.any() and not val.any() and not wire.any() and bool((x == 1).all())


def test_an_older_extension_is_gone_without(monkeypatch):
    import sys
    import types

    import paper_2410_12707_amd as package

    older = types.ModuleType(package.__name__ + "._marshal")  # it read the arrays of the segmented calls and made no call
    older.tensors = older.int64s = lambda *_: None
    monkeypatch.setitem(sys.modules, older.__name__, older)
    monkeypatch.setattr(package, "_marshal", older, raising=False)
    monkeypatch.setattr(B, "_marshal", None)
    x, idx, val, ws = torch.zeros(64), torch.zeros(8, dtype=torch.int32), torch.zeros(8), torch.zeros(256, dtype=torch.uint8)
    with pytest.warns(RuntimeWarning, match="older source"):
        with pytest.raises(ValueError):  # what the call in Python says of host memory
            B.adatopk_compress(x, 8, idx, val, None, ws)
    assert B._marshal is False
