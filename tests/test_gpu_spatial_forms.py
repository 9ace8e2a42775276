"""Every table size and workgroup size of spatial_frames_kernel that a variant of the rule reaches (many short frames take four
wavefronts, few of them sixteen), labels that share their low or their high bits, against the oracle, 0 differing bits."""
import numpy as np
import pytest

from test_gpu_spatial_variants import batch, check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nms():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2502_00535_amd.binding as binding

    return binding


@pytest.mark.parametrize("frames,n", [(1, 1), (1, 64), (46, 256), (256, 40), (257, 40), (600, 20), (3000, 4), (1, 257), (22, 270), (12, 500)])
def test_short_frames(nms, oracle, frames, n):
    print(f"case {frames} x {n}", flush=True)
    data = batch(frames + n, frames, n)
    for measure in ("iou", "outranking_area"):
        for labelled in (True, False):
            check(nms, oracle, data, 0.45, dict(rule="paper", measure=measure, compare="gt", ties="index", pixel_offset=1.0, labelled=labelled))


@pytest.mark.parametrize("frames,n", [(2, 2300), (2, 4096), (4, 2049), (9, 1025), (6, 1640), (7, 1350)])
def test_shapes_at_the_lines(nms, oracle, frames, n):
    """The smallest batches of frames of their length that are put in order of place (up to 64 workgroups per frame)."""
    from test_gpu_spatial_frames import check as check_default

    print(f"case {frames} x {n}", flush=True)
    boxes, scores, _, counts = batch(n, frames, n)
    check_default(nms, oracle, boxes, scores, 0.45)
    check_default(nms, oracle, boxes, scores, 0.3, counts)


@pytest.mark.parametrize("frames,n", [(3, 250), (3, 1000), (3, 2500)])
def test_labels_by_their_bits(nms, oracle, frames, n):
    """The bin of a label comes from eight bits of it: labels equal in four of them, in all eight, and with the sign bit."""
    boxes, scores, _, counts = batch(n, frames, n)
    rng = np.random.default_rng(n)
    opts = dict(rule="paper", measure="iou", compare="ge", ties="index", pixel_offset=1.0, labelled=True)
    for labels in (16 * rng.integers(0, 16, (frames, n)), rng.integers(0, 16, (frames, n)), 17 * rng.integers(0, 16, (frames, n)),
                   256 * rng.integers(0, 5, (frames, n)) + 3, rng.integers(0, 256, (frames, n)), rng.integers(-2, 2, (frames, n)) * 2 ** 30):
        check(nms, oracle, (boxes, scores, labels.astype(np.int32), counts), 0.4, opts)
