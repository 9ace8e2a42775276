"""The native marshalling leaves every argument that is not in order to the Python path, which names it; no GPU needed."""
import os

import numpy as np
import pytest
import torch


def test_what_is_not_in_order_is_named():
    import paper_2502_00535_amd.binding as nms

    n = 8
    boxes, scores = torch.zeros(1, n, 4), torch.zeros(1, n)
    keep, ws = torch.zeros(1, n, dtype=torch.uint8), torch.zeros(1 << 16, dtype=torch.uint8)
    run = nms._marshal.run
    good = [nms._RUN_BATCHED, boxes, scores, None, n, 1, 0.5, keep, ws, None]
    assert run(*good) is None                                     # tensors of the CPU
    for at, other in ((1, "boxes"), (1, None), (3, 5), (4, -1), (4, 1 << 40), (4, 8.0), (5, True), (6, 1), (8, None)):
        assert run(*(good[:at] + [other] + good[at + 1:])) is None
    with pytest.raises(TypeError):
        run(*good[:-1])
    for call, args in ((nms.nms_run_ws, (boxes, scores, n, 0.5, keep, None)), (nms.nms_run_batched, (boxes, scores, None, n, 1, 0.5, keep, None)),
                       (nms.nms_run_ranked_batched, (boxes, scores, None, n, 1, 0.5, keep, None)),
                       (nms.nms_run_greedy_batched, (boxes, scores, None, n, 1, 0.5, keep, None))):
        with pytest.raises(ValueError, match="boxes: tensor must live on the GPU"):
            call(*args)
        with pytest.raises(TypeError, match="boxes: expected a torch tensor"):
            call("boxes", *args[1:])


def test_without_the_native_module():
    """A Python that the module was not built for, or a machine without a C compiler: the package imports, and every call is
    marshalled (and refused) as before."""
    import subprocess
    import sys

    code = """
import sys
sys.modules["paper_2502_00535_amd._marshal"] = None
import torch
import paper_2502_00535_amd.binding as nms
assert nms._marshal is None
boxes, scores, keep = torch.zeros(1, 8, 4), torch.zeros(1, 8), torch.zeros(1, 8, dtype=torch.uint8)
for call, args in ((nms.nms_run_ws, (boxes, scores, 8, 0.5, keep, None)), (nms.nms_run_batched, (boxes, scores, None, 8, 1, 0.5, keep, None)),
                   (nms.nms_run_ranked_batched, (boxes, scores, None, 8, 1, 0.5, keep, None)),
                   (nms.nms_run_greedy_batched, (boxes, scores, None, 8, 1, 0.5, keep, None))):
    try:
        call(*args)
    except ValueError as e:
        assert "boxes: tensor must live on the GPU" in str(e)
    else:
        raise AssertionError(call)
    try:
        call("boxes", *args[1:])
    except TypeError as e:
        assert "boxes: expected a torch tensor" in str(e)
    else:
        raise AssertionError(call)
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    proc = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr[-2000:]


def test_library_builds_without_a_c_compiler(monkeypatch, tmp_path):
    from paper_2502_00535_amd import build

    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.so"))
    monkeypatch.setenv("CC", "/nonexistent/cc")
    (tmp_path / "_marshal.so").write_bytes(b"of an earlier state")
    with pytest.warns(UserWarning, match="native marshalling not built"):
        assert build.build_marshal_if_possible() is None
    assert not (tmp_path / "_marshal.so").exists()


class Claimed(torch.Tensor):
    """A tensor that says of itself what the native path asks for (no GPU, nothing is read): `count` elements on one."""
    count = 1
    is_cuda = True

    def numel(self):
        return self.count


def claimed(dtype, count):
    t = torch.zeros(1, dtype=dtype).as_subclass(Claimed)
    t.count = count
    return t


def test_sizes_are_bounded_before_they_are_multiplied():
    """The boxes' element count is 4 n_max frames: near 2^31 each, that product passes 2^63 (it once wrapped to a negative number, which
    no tensor is too small for).  Sizes the library refuses are left to the other path; what fits goes through."""
    import ctypes

    import paper_2502_00535_amd.binding as nms

    calls = []
    proto = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * 3, ctypes.c_int, ctypes.c_int, ctypes.c_float, *[ctypes.c_void_p] * 2,
                             ctypes.c_size_t, ctypes.c_void_p)
    fn = proto(lambda *a: calls.append(a[3:6]) or 0)
    address = ctypes.cast(fn, ctypes.c_void_p).value

    class Stream:
        cuda_stream = 0

    def run(n, f, boxes):
        many = 2 ** 62 + 2 ** 61
        return nms._marshal.run(address, claimed(torch.float32, boxes), claimed(torch.float32, many), None, n, f, 0.5,
                                claimed(torch.uint8, many), claimed(torch.uint8, many), Stream())

    assert run(8, 2, 64) == 0 and run(8, 2, 63) is None
    assert run(65536, 65535, 4 * 65536 * 65535) == 0 and run(65536, 65535, 4 * 65536 * 65535 - 1) is None
    for n, f in ((2 ** 31 - 1, 2 ** 31 - 1), (2 ** 31 - 1, 2 ** 30 + 1), (65537, 1), (1, 65536)):
        assert run(n, f, 1) is None, (n, f)
    assert [c[:2] for c in calls] == [(8, 2), (65536, 65535)]


@pytest.mark.gpu
def test_the_two_paths_agree():
    import paper_2502_00535_amd.binding as nms

    n = 300
    g = torch.Generator().manual_seed(1)
    xy = torch.rand(2, n, 2, generator=g) * 200
    boxes, scores = torch.cat([xy, xy + 30], -1).cuda(), torch.rand(2, n, generator=g).cuda()
    ws = torch.empty(nms.nms_workspace_bytes(n, 2), dtype=torch.uint8, device="cuda")
    a, b, c = (torch.full((2, n), 9, dtype=torch.uint8, device="cuda") for _ in range(3))
    nms.nms_run_batched(boxes, scores, None, n, 2, 0.5, a, ws)
    nms.nms_run_batched(boxes, scores, None, n, 2, np.float32(0.5), b, ws)  # not a float: the Python path
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    nms.nms_run_batched(boxes, scores, None, n, 2, 0.5, c, ws, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c) and int(a.max()) == 1
    for bad in (boxes.double(), boxes[:, ::2], boxes[:1], boxes.cpu()):
        with pytest.raises((TypeError, ValueError)):
            nms.nms_run_batched(bad, scores, None, n, 2, 0.5, a, ws)
    with pytest.raises(nms.NmsError):
        nms.nms_run_batched(boxes, scores, None, n, 2, 0.5, a, ws[:256])
