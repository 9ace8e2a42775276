"""The greedy rule with labels on large batches: every class by a wavefront of its own, frames with a class that
is a large share of the frame walked by the whole workgroup, against the oracle.  Bar: 0 differing keep bits."""
import numpy as np
import pytest

from workloads import random_frame

from test_gpu_variants import ExFrames, nms, oracle_ex  # noqa: F401  (nms: fixture)
from test_host_logic import largest_bin

pytestmark = pytest.mark.gpu


def labels_of(kind, rng, n):
    if kind == "twenty":
        return rng.integers(0, 20, n)
    if kind == "one":
        return np.zeros(n, np.int64)
    if kind == "largest_bin":  # 1024 boxes of one label: the most that a wavefront takes, in a frame of 4096
        return rng.permutation(np.where(np.arange(n) < 1024, 3, 4 + np.arange(n) % 90))
    if kind == "one_more":
        return rng.permutation(np.where(np.arange(n) < 1025, 3, 4 + np.arange(n) % 90))
    if kind == "last_bin":  # the bin behind which the places without a box stand
        return np.where(rng.random(n) < 0.3, 255, rng.integers(0, 300, n))
    # several labels per bin, any 32-bit value
    return rng.choice(np.array([-2 ** 31, 2 ** 31 - 1, -1, 0, 0x101, 0x10001, 0x10100, 1, 257]), n)


@pytest.mark.parametrize("n_max,frames", [(64, 2048), (1024, 128), (1025, 128), (4096, 33)])
def test_labels(nms, oracle, n_max, frames):  # noqa: F811
    rng = np.random.default_rng(n_max)
    kinds = ["twenty", "one", "largest_bin", "one_more", "last_bin", "any"]
    distinct = 12
    boxes = np.zeros((distinct, n_max, 4), np.float32)
    scores = np.zeros((distinct, n_max), np.float32)
    classes = np.zeros((distinct, n_max), np.int32)
    counts = np.zeros(distinct, np.int32)
    for f in range(distinct):
        boxes[f], scores[f] = random_frame(77 * n_max + f, n_max, extent=300 + 60 * f, max_side=120, integer=f % 2 == 0,
                                           score_levels=(0, 40)[f % 2])
        classes[f] = labels_of(kinds[f % 6], rng, n_max).astype(np.int32)
        counts[f] = n_max if f < 6 else [0, 1, 63, 64, n_max - 1, n_max // 2][f - 6]
    which = np.arange(frames) % distinct
    for ragged in (False, True):
        dev = ExFrames(nms, boxes[which], scores[which], classes[which], counts[which] if ragged else None)
        for measure, compare, ties, offset in (("iou", "gt", "index", 0.0), ("iou", "ge", "ignore", 1.0),
                                               ("outranking_area", "gt", "ignore", 0.0), ("outranking_area", "ge", "index", 1.0)):
            opts = dict(rule="greedy", measure=measure, compare=compare, ties=ties, pixel_offset=offset, labelled=True)
            print(f"case n_max={n_max} frames={frames} ragged={ragged} {opts}", flush=True)
            want = oracle_ex(oracle, boxes, scores, classes, 0.45, opts, counts if ragged else None, workers=8)[which]
            got = dev.run(0.45, opts)
            assert np.array_equal(got, want), f"{opts}: {(got != want).sum()} differing keep bits"


# Every kernel (4, 8 and 16 wavefronts, tables of 256 to 4096 boxes) at the ends of its range, in frames whose largest bin
# is at the bound and one beyond, the longest that are always walked, and lengths around whole tiles.
@pytest.mark.parametrize("n_max,frames", [(64, 2048), (192, 769), (193, 769), (256, 769), (257, 769), (512, 769), (513, 769), (1024, 769),
                                          (171, 768), (512, 768), (513, 768), (1024, 129), (1025, 128), (1800, 80), (4096, 33)])
def test_bins_at_the_bound(nms, oracle, n_max, frames):  # noqa: F811
    rng = np.random.default_rng(n_max)
    counts = np.minimum(n_max, [n_max, n_max, n_max - 1, n_max // 2, 193, 320, 65, 64, 1, 0]).astype(np.int32)
    distinct = len(counts)
    boxes = np.zeros((distinct, n_max, 4), np.float32)
    scores = np.zeros((distinct, n_max), np.float32)
    classes = np.zeros((distinct, n_max), np.int32)
    for f in range(distinct):
        boxes[f], scores[f] = random_frame(31 * n_max + f, n_max, extent=250 + 50 * f, max_side=120, integer=f % 2 == 0,
                                           score_levels=(0, 40)[f % 2])
        c = int(counts[f])
        rows = largest_bin(c) + f % 2
        classes[f, :c] = rng.permutation(np.where(np.arange(c) < rows, 7, 8 + np.arange(c) % 60))
    which = np.arange(frames) % distinct
    dev = ExFrames(nms, boxes[which], scores[which], classes[which], counts[which])
    for measure, compare, ties, offset in (("iou", "gt", "index", 0.0), ("outranking_area", "ge", "ignore", 1.0)):
        opts = dict(rule="greedy", measure=measure, compare=compare, ties=ties, pixel_offset=offset, labelled=True)
        print(f"case n_max={n_max} frames={frames} {opts}", flush=True)
        want = oracle_ex(oracle, boxes, scores, classes, 0.45, opts, counts, workers=8)[which]
        got = dev.run(0.45, opts)
        assert np.array_equal(got, want), f"{opts}: {(got != want).sum()} differing keep bits"


@pytest.mark.parametrize("n,frames", [(640, 205), (1024, 128)])
def test_one_label_costs_little_more_than_none(nms, n, frames):  # noqa: F811
    """All boxes of one label are one bin: as one wavefront's chain 3 to 5 times the unlabelled call, walked about
    1.2 to 1.5 times.  The bound lies between, well beyond what a run's times differ."""
    import torch

    dev = torch.device("cuda:0")
    frame = random_frame(3, n, extent=2000, max_side=120, integer=False, score_levels=0)
    boxes = torch.from_numpy(np.tile(frame[0], (frames, 1, 1))).to(dev)
    scores = torch.from_numpy(np.tile(frame[1], (frames, 1))).to(dev)
    keep = torch.empty((2, frames, n), dtype=torch.uint8, device=dev)
    ws = torch.empty(nms.nms_ex_workspace_bytes(n, frames), dtype=torch.uint8, device=dev)
    ones = torch.ones((frames, n), dtype=torch.int32, device=dev)
    times = [[], []]
    for _ in range(6):
        for i, classes in enumerate((None, ones)):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(20):
                nms.nms_run_ex_batched(boxes, scores, None, n, frames, 0.5, keep[i], ws, rule="greedy", measure="iou",
                                       compare="gt", pixel_offset=0.0, classes=classes)
            end.record()
            end.synchronize()
            times[i].append(begin.elapsed_time(end) / 20)
    assert torch.equal(keep[0], keep[1])
    plain, labelled = (min(t) for t in times)
    print(f"n={n} frames={frames}: {1e3 * plain:.1f} us without labels, {1e3 * labelled:.1f} us with one", flush=True)
    assert labelled < 2.0 * plain
