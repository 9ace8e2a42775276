"""The greedy rule under IoU in order of place (place_relation_kernel, place_resolve_kernel) on frames whose boxes crowd: rows with
eliminators in more tiles than are written down, frames that are walked after the rounds, frames of more than 4096 boxes that
the general kernels finish, next to frames that need none of it; 0 differing bits against the oracle.  And such frames take no multiple of
the time of others."""
import itertools

import numpy as np
import pytest

from test_gpu_variants import ExFrames, oracle_ex
from workloads import clustered_frame, random_frame

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nms():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2502_00535_amd.binding as binding

    return binding


def objects_frame(seed, n, objects):
    """n candidates around few objects: thousands of boxes that touch."""
    b, s = clustered_frame(seed, objects=objects, width=3840, height=2160, size_lo=150.0, size_hi=500.0, per_object=-(-n // objects))
    return b[:n], s[:n]


def chain_frame(seed, n, step=4.0, side=10.0):
    """Boxes in a line, each eliminating the next few; scores fall along the line, input order random for odd seeds."""
    x = np.arange(n, dtype=np.float32) * np.float32(step)
    b = np.stack([x, np.zeros(n, np.float32), x + side, np.full(n, side, np.float32)], 1)
    s = (1.0 - np.arange(n) / n).astype(np.float32)
    p = np.random.default_rng(seed).permutation(n) if seed % 2 else np.arange(n)
    return b[p], s[p]


def mixed_frame(seed, n):
    """One object with half of the boxes, the rest spread."""
    b0, s0 = objects_frame(seed, n // 2, 1)
    b1, s1 = random_frame(seed, n - n // 2, extent=6000, max_side=80, integer=False)
    p = np.random.default_rng(seed).permutation(n)
    return np.concatenate([b0, b1])[p], np.concatenate([s0, s1])[p]


SCENES = {"objects1": lambda f, n: objects_frame(f, n, 1), "objects4": lambda f, n: objects_frame(f, n, 4), "objects16": lambda f, n: objects_frame(f, n, 16),
          "mixed": mixed_frame, "chain": chain_frame, "slide": lambda f, n: chain_frame(f, n, 5.0, 100.0),
          "spread": lambda f, n: random_frame(f, n, extent=9000, max_side=90, integer=False),
          "copies": lambda f, n: (np.repeat(random_frame(f, n // 50 + 1, extent=900, max_side=90)[0], 50, 0)[:n], np.float32(0.5) + 0 * random_frame(f, n)[1])}


@pytest.mark.parametrize("frames,n", [(8, 2049), (8, 3000), (16, 4096), (8, 4097), (8, 8192)])
def test_crowded_frames(nms, oracle, frames, n):
    """A scene of every kind in one call, with and without labels and ties."""
    print(f"case {frames} x {n}", flush=True)
    kinds = [SCENES[k](f, n) for f, k in zip(range(frames), itertools.cycle(SCENES))]
    boxes, scores = np.stack([k[0] for k in kinds]).astype(np.float32), np.stack([k[1] for k in kinds]).astype(np.float32)
    rng = np.random.default_rng(n)
    scores[2] = np.round(scores[2] * 40) / 40
    labels = rng.integers(0, 2, (frames, n)).astype(np.int32)
    counts = np.full(frames, n, np.int32)
    counts[1:4] = [n - 1, 0, 2048]
    for (ties, labelled), theta in itertools.product((("index", False), ("ignore", False), ("index", True)), (0.5, 0.1)):
        opts = dict(rule="greedy", measure="iou", compare="gt", ties=ties, pixel_offset=1.0, labelled=labelled)
        for c in (None, counts):
            want = oracle_ex(oracle, boxes, scores, labels, theta, opts, c, workers=16)
            got = ExFrames(nms, boxes, scores, labels, c).run(theta, opts)
            assert np.array_equal(got, want), f"{(got != want).sum(axis=1)} differing keep bits per frame: {opts} {theta}"


@pytest.mark.parametrize("frames,n,objects", [(31, 4096, 1), (31, 4096, 6), (6, 4096, 40), (7, 4096, 40), (40, 5000, 1)])
def test_batches_of_crowded_frames(nms, oracle, frames, n, objects):
    """More workgroups than fit at once: later tiles of a frame are not related once many of its rows are crowded."""
    print(f"case {frames} x {n} x {objects}", flush=True)
    kinds = [objects_frame(f + n, n, objects) for f in range(frames)]
    boxes, scores = np.stack([k[0] for k in kinds]), np.stack([k[1] for k in kinds])
    labels = np.zeros((frames, n), np.int32)
    opts = dict(rule="greedy", measure="iou", compare="ge", ties="index", pixel_offset=0.0, labelled=False)
    want = oracle_ex(oracle, boxes, scores, labels, 0.5, opts, None, workers=16)
    dev = ExFrames(nms, boxes, scores, labels)
    for _ in range(2):
        got = dev.run(0.5, opts)
        assert np.array_equal(got, want), f"{(got != want).sum(axis=1)} differing keep bits per frame"


@pytest.mark.parametrize("n", [4096, 8000])
def test_crowded_frames_take_no_multiple_of_the_time(nms, n):
    """Where thousands of candidates crowd around one object, or a chain of eliminators is long, the call once took seventy times
    as long as on spread clusters; the general kernels would take 1.1 to 5 times as long."""
    import torch

    def us(b, s):
        dev = ExFrames(nms, b[None], s[None], np.zeros((1, n), np.int32))
        opts = dict(rule="greedy", measure="iou", compare="gt", pixel_offset=0.0)
        call = lambda: nms.nms_run_ex_batched(dev.boxes, dev.scores, None, n, 1, 0.5, dev.keep, dev.ws, **opts)
        call()
        best = 1e9
        for _ in range(5):
            a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                call()
            z.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(z) * 100)
        return best

    b, s = clustered_frame(1, objects=(n + 15) // 16, width=3840, height=2160, size_lo=24.0, size_hi=384.0)
    usual = us(b[:n], s[:n])
    for name, bound in (("objects1", 6), ("objects4", 6), ("objects16", 6), ("mixed", 8), ("slide", 12)):
        crowded = us(*SCENES[name](0, n))
        print(f"{n} {name}: {crowded:.1f} us, clusters {usual:.1f}", flush=True)
        assert crowded < bound * usual, f"{name}: {crowded:.1f} us against {usual:.1f}"
