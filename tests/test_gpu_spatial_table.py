"""Frames of more than 4096 boxes in order of place (place_sort_kernel, place_scan_kernel, what nms_run_batched takes for them)
against the oracle's plain double loop, 0 differing bits: every number of boxes per thread, several chunks of boxes per
workgroup, shares of one to sixteen tiles, cells that a share cuts, places that are all the same or far apart, ties, ragged batches."""
import numpy as np
import pytest

from gpu_util import DeviceFrames, oracle_keep_frames
from workloads import clustered_frame, random_frame

pytestmark = pytest.mark.gpu


def check(oracle, boxes, scores, theta, counts=None):
    import paper_2502_00535_amd.binding as nms

    want = oracle_keep_frames(oracle, boxes, scores, np.float32(theta), counts)
    dev = DeviceFrames(nms, boxes, scores, counts)
    for _ in range(2):
        got = dev.fused(float(theta))
        assert np.array_equal(got, want), f"{(got != want).sum()} differing keep bits"
    return want


@pytest.mark.parametrize("frames,n", [(1, 4097), (1, 8192), (1, 8193), (2, 6000), (1, 16384), (1, 16385), (1, 40000), (9, 5001), (40, 4500), (70, 4160)])
def test_shapes(oracle, frames, n):
    print(f"case {frames} x {n}", flush=True)
    fr = [clustered_frame(n + f, objects=(n + 15) // 16, width=3840, height=2160, size_lo=16.0, size_hi=300.0) for f in range(frames)]
    boxes, scores = np.stack([x[0][:n] for x in fr]), np.stack([x[1][:n] for x in fr])
    counts = None
    if frames > 1:
        counts = np.random.default_rng(n).integers(0, n + 1, frames).astype(np.int32)
        counts[:2] = [n, [0, 1, 64, 4097][frames % 4]]
    assert check(oracle, boxes, scores, [0.5, 0.3][n % 2], counts).sum() > 0


def test_places(oracle):
    n = 9000
    for kind in range(5):
        print(f"case {kind}", flush=True)
        rng = np.random.default_rng(kind)
        b, s = random_frame(kind, n, extent=2500, max_side=70, integer=kind % 2 == 0, score_levels=2000)
        if kind == 0:
            b[:] = np.array([5, 5, 40, 30], np.float32)      # one place
        elif kind == 1:                                      # two cells hold almost all: every share cuts one
            b[:, :2] = np.where(rng.random((n, 1)) < 0.5, 100.0, 900.0) + rng.random((n, 2))
            b[:, 2:] = b[:, :2] + 9
            b[:3, 2:] += 2000
        elif kind == 2:                                      # a few far away
            b[rng.permutation(n)[:7]] += np.float32(1e7)
        elif kind == 3:                                      # every size
            b[:, 2:] = b[:, :2] + np.exp2(rng.uniform(-6, 11, n)).astype(np.float32)[:, None]
        else:                                                # equal scores, copies
            s[:] = 0.5
            b[rng.integers(0, n, n // 2)] = b[rng.integers(0, n, n // 2)]
        for theta in (0.5, 2.0 ** -40, 1.0):
            check(oracle, b[None], s[None], theta)
