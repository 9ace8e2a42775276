"""The greedy rule with labels on large batches: every class by a wavefront of its own, frames with a
class beyond 1024 boxes by the walk, against the oracle.  Bar: 0 differing keep bits."""
import numpy as np
import pytest

from workloads import random_frame

from test_gpu_variants import ExFrames, nms, oracle_ex  # noqa: F401  (nms: fixture)

pytestmark = pytest.mark.gpu


def labels_of(kind, rng, n):
    if kind == "twenty":
        return rng.integers(0, 20, n)
    if kind == "one":
        return np.zeros(n, np.int64)
    if kind == "largest_bin":  # 1024 boxes of one label: the most that a wavefront takes
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
