"""The paper's rule with IoU, strict compare, ignored ties and labels in order of place (spatial_frames_kernel, place_sort_kernel and
place_scan_kernel with the variants), the greedy rule under IoU in order of
place (place_relation_kernel, place_resolve_kernel) and on short frames (greedy_small_kernel), against the oracle, 0 differing
bits: every table size, labels in and outside 0 .. 255 and in one bin, boxes without area, ties between copies, frame lengths around
tiles, thresholds with and without a division-free form."""
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


def batch(seed, frames, n, offset0=False):
    rng = np.random.default_rng(seed)
    boxes, scores, labels = np.zeros((frames, n, 4), np.float32), np.zeros((frames, n), np.float32), np.zeros((frames, n), np.int32)
    for f in range(frames):
        if f % 2:
            b, s = clustered_frame(seed + f, objects=(n + 15) // 16, width=1920, height=1080, size_lo=16.0, size_hi=300.0)
            b, s = b[:n], s[:n]
        else:
            b, s = random_frame(seed + f, n, extent=900, max_side=80, integer=f % 4 == 0, score_levels=max(3, n // 4))
        src, dst = rng.integers(0, n, n // 8), rng.integers(0, n, n // 8)
        b[dst], s[dst] = b[src], s[src]
        boxes[f], scores[f] = b, s
        labels[f] = [rng.integers(0, 5, n), rng.integers(0, 20, n), 16 * rng.integers(0, 9, n), rng.integers(-3, 400, n), np.full(n, 7)][f % 5]
    if offset0:  # continuous coordinates: extents above 0
        boxes[..., 2:] += np.float32(1.0)
    counts = rng.integers(0, n + 1, frames).astype(np.int32)
    counts[0] = n
    return boxes, scores, labels, counts


def check(nms, oracle, data, theta, opts):
    boxes, scores, labels, counts = data
    want = oracle_ex(oracle, boxes, scores, labels, theta, opts, counts, workers=16)
    dev = ExFrames(nms, boxes, scores, labels, counts)
    got = dev.run(theta, opts)
    assert np.array_equal(got, want), f"{(got != want).sum()} differing keep bits: {opts}"


@pytest.mark.parametrize("frames,n", [(9, 100), (40, 256), (10, 300), (6, 512), (11, 1000), (5, 1025), (6, 2048), (5, 2049), (7, 4096), (2, 4097), (3, 9000)])
def test_papers_rule(nms, oracle, frames, n):
    for measure, compare, ties, labelled in itertools.product(("iou", "outranking_area"), ("ge", "gt"), ("index", "ignore"), (False, True)):
        opts = dict(rule="paper", measure=measure, compare=compare, ties=ties, pixel_offset=1.0 if compare == "ge" or measure != "iou" else 0.0,
                    labelled=labelled)
        print(f"case {frames} x {n} {opts}", flush=True)
        check(nms, oracle, batch(n, frames, n, offset0=opts["pixel_offset"] == 0.0), 0.45, opts)


def test_equal_iou_at_the_threshold(nms, oracle):
    """Pairs whose quotient is the threshold exactly, where the compare decides."""
    n = 1500
    base = np.zeros((n, 4), np.float32)
    cell = np.arange(n)
    base[:, 0], base[:, 1] = (cell % 40) * 64.0, (cell // 40) * 64.0
    base[:, 2:] = base[:, :2] + 32.0
    base[1::2, :2] = base[:-1:2, :2]
    base[1::2, 2:] = base[:-1:2, :2] + np.array([32.0, 16.0], np.float32)   # IoU 1/2 with offset 0
    scores = np.random.default_rng(1).permutation(n).astype(np.float32)[None]
    labels = np.zeros((1, n), np.int32)
    for compare, labelled in itertools.product(("ge", "gt"), (False, True)):
        opts = dict(rule="paper", measure="iou", compare=compare, ties="index", pixel_offset=0.0, labelled=labelled)
        check(nms, oracle, (base[None], scores, labels, np.array([n], np.int32)), 0.5, opts)


@pytest.mark.parametrize("frames,n", [(3, 1), (5, 63), (5, 64), (7, 65), (40, 128), (9, 129), (30, 191), (300, 192), (9, 193)])
def test_greedy_on_short_frames(nms, oracle, frames, n):
    print(f"case {frames} x {n}", flush=True)
    for measure, compare, ties, labelled in itertools.product(("outranking_area", "iou"), ("ge", "gt"), ("index", "ignore"), (False, True)):
        opts = dict(rule="greedy", measure=measure, compare=compare, ties=ties, pixel_offset=1.0 if compare == "ge" else 0.0, labelled=labelled)
        data = batch(7 * n, frames, n, offset0=compare == "gt")
        for theta in (0.4, 0.0):
            check(nms, oracle, data, theta, opts)


@pytest.mark.parametrize("frames,n", [(1, 257), (1, 1000), (3, 2000), (2, 2049), (3, 4096), (2, 4097), (1, 8192), (1, 8193)])
def test_greedy_iou(nms, oracle, frames, n):
    print(f"case {frames} x {n}", flush=True)
    for compare, ties, labelled in itertools.product(("ge", "gt"), ("index", "ignore"), (False, True)):
        opts = dict(rule="greedy", measure="iou", compare=compare, ties=ties, pixel_offset=1.0 if compare == "ge" else 0.0, labelled=labelled)
        check(nms, oracle, batch(5 * n, frames, n, offset0=compare == "gt"), 0.45, opts)


def test_greedy_iou_chains_and_crowds(nms, oracle):
    """Long chains of boxes that eliminate only the next one (many rounds), and boxes with eliminators in every tile (more masks per row
    than are kept in registers)."""
    opts = dict(rule="greedy", measure="iou", compare="gt", ties="index", pixel_offset=0.0, labelled=False)
    n = 3000
    step = np.arange(n, dtype=np.float32) * 4
    chain = np.stack([step, np.zeros(n, np.float32), step + 10, np.full(n, 10, np.float32)], 1)
    scores = (1.0 - np.arange(n) / n).astype(np.float32)
    labels, counts = np.zeros((1, n), np.int32), np.array([n], np.int32)
    perm = np.random.default_rng(1).permutation(n)
    check(nms, oracle, (chain[None, perm], scores[None, perm], labels, counts), 0.3, opts)
    rng = np.random.default_rng(2)
    for n in (2500, 6000):
        xy = rng.random((1, n, 2)).astype(np.float32) * 300
        boxes = np.concatenate([xy, xy + 100 + 50 * rng.random((1, n, 2)).astype(np.float32)], -1)
        data = (boxes, rng.random((1, n)).astype(np.float32), np.zeros((1, n), np.int32), np.array([n], np.int32))
        for theta in (0.02, 0.3, 0.6):
            check(nms, oracle, data, theta, opts)
