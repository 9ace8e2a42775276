"""Frames in order of place (spatial_frames_kernel, what nms_run_batched takes for most batches of frames of
449 to 4096 boxes) against the oracle's plain double loop, 0 differing bits: every number of wavefronts
per tile of victims and every table size, frame lengths around tiles and table sizes, boxes of all size classes and at
the border of the grid, places that are all the same, far outside the sampled range or in one line, frames without boxes."""
import numpy as np
import pytest

from gpu_util import DeviceFrames, oracle_keep_frames
from workloads import anchor_frame, clustered_frame, random_frame, scores_of_every_kind

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nms():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2502_00535_amd.binding as binding

    return binding


def check(nms, oracle, boxes, scores, theta, counts=None):
    want = oracle_keep_frames(oracle, boxes, scores, np.float32(theta), counts)
    dev = DeviceFrames(nms, boxes, scores, counts)
    for _ in range(2):  # the order inside a cell differs from call to call
        got = dev.fused(float(theta))
        assert np.array_equal(got, want), f"{(got != want).sum()} differing keep bits"
    return want


# workgroups per frame 1 .. 64, wavefronts per tile of victims 1, 2, 4; 512, 1024, 2048 and 4096 rows
SHAPES = [(512, 449), (512, 512), (300, 513), (28, 1000), (60, 700), (130, 1024), (257, 640), (8, 1025), (30, 1537), (130, 2048),
          (260, 1100), (2, 2049), (3, 3000), (5, 4095), (20, 4096), (130, 2500)]


@pytest.mark.parametrize("frames,n", SHAPES)
def test_shapes(nms, oracle, frames, n):
    print(f"case {frames} x {n}", flush=True)
    fr = [clustered_frame(7 * f + n, objects=(n + 15) // 16, width=1920, height=1080, size_lo=16.0, size_hi=400.0) if f % 2 else anchor_frame(f, n)
          for f in range(frames)]
    boxes, scores = np.stack([x[0][:n] for x in fr]), np.stack([x[1][:n] for x in fr])
    rng = np.random.default_rng(n)
    counts = rng.integers(0, n + 1, frames).astype(np.int32)
    some = [n, 0, 1, 2, 63, 64, 65, n - 1]
    counts[:len(some)] = some[:frames]
    assert check(nms, oracle, boxes, scores, 0.45).sum() > 0
    check(nms, oracle, boxes, scores, [0.3, 0.7][n % 2], counts)


@pytest.mark.parametrize("frames,n", [(40, 1024), (3, 4096), (300, 1300)])
def test_places(nms, oracle, frames, n):
    """What a grid over 64 sampled centres can meet."""
    print(f"case {frames} x {n}", flush=True)
    kinds = []
    for f in range(frames):
        rng = np.random.default_rng(100 * n + f)
        b, s = random_frame(f + n, n, extent=900, max_side=70, integer=f % 2 == 0, score_levels=max(3, n // 5))
        kind = f % 10
        if kind == 0:                                   # one place
            b[:] = np.array([5, 5, 40, 30], np.float32)
        elif kind == 1:                                 # one line
            b[:, 1], b[:, 3] = 10.0, 50.0
        elif kind == 2:                                 # a few far away, seldom sampled
            far = rng.permutation(n)[:9]
            b[far] += np.float32(1e6)
            b[rng.permutation(n)[:5]] -= np.float32(3e5)
        elif kind == 3:                                 # every size from a point to the whole picture
            side = np.exp2(rng.uniform(-6, 11, n)).astype(np.float32)
            b[:, 2:] = b[:, :2] + side[:, None]
        elif kind == 4:                                 # one cell holds almost all
            b[10:, :2] = 100 + rng.random((n - 10, 2)).astype(np.float32)
            b[10:, 2:] = b[10:, :2] + 20
        elif kind == 5:                                 # touching and one-pixel boxes on the lattice
            b[:, :2] = np.floor(b[:, :2] / 8) * 8
            b[:, 2:] = b[:, :2] + 7
        elif kind == 6:                                 # normalised coordinates
            b /= np.float32(900)
        elif kind == 7:                                 # large coordinates
            b *= np.float32(2.0 ** 20)
        elif kind == 8:                                 # input sorted by score
            s = np.sort(s)[::-1].copy()
        else:
            s = scores_of_every_kind(f, n)
        kinds.append((b, s))
    boxes, scores = np.stack([k[0] for k in kinds]), np.stack([k[1] for k in kinds])
    for theta in (0.5, 0.05, 1.0, 2.0 ** -40, 3.0):
        check(nms, oracle, boxes, scores, theta)


def test_equal_scores_and_copies(nms, oracle):
    """Every tie is decided by the index, between copies of a box in particular."""
    for frames, n in ((64, 1000), (2, 4000), (512, 500)):
        print(f"case {frames} x {n}", flush=True)
        rng = np.random.default_rng(n)
        boxes = np.stack([random_frame(f, n, extent=1500, max_side=90)[0] for f in range(frames)])
        src, dst = rng.integers(0, n, n // 2), rng.integers(0, n, n // 2)
        boxes[:, dst] = boxes[:, src]
        check(nms, oracle, boxes, np.full((frames, n), 0.25, np.float32), 0.5)
        check(nms, oracle, boxes, rng.integers(0, 3, (frames, n)).astype(np.float32), 0.4)


def test_can_be_captured(nms, oracle):
    """One kernel and nothing else: replays with other inputs in the same buffers."""
    import torch

    frames, n = 64, 1024
    sets = [np.stack([x[k] for x in [clustered_frame(50 * i + f, 64, 1920, 1080, 32.0, 256.0) for f in range(frames)]])
            for i in range(3) for k in (0, 1)]
    dev = DeviceFrames(nms, sets[0], sets[1])
    dev.fused(0.5)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nms.nms_run_batched(dev.boxes, dev.scores, None, n, frames, 0.5, dev.keep, dev.run_ws)
    for i in (1, 2, 0, 1):
        dev.boxes.copy_(torch.from_numpy(sets[2 * i]))
        dev.scores.copy_(torch.from_numpy(sets[2 * i + 1]))
        dev.keep.fill_(9)
        graph.replay()
        torch.cuda.synchronize()
        want = oracle_keep_frames(oracle, sets[2 * i], sets[2 * i + 1], np.float32(0.5))
        assert np.array_equal(dev.keep.cpu().numpy(), want)
