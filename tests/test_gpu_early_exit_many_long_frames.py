"""More than 128 frames of more than 4096 boxes through nms_run_early_exit_batched and nms_run_batched: a workgroup per frame would do for
so many, but a frame beyond 4096 boxes does not fit one."""
import numpy as np
import pytest

from gpu_util import DeviceFrames, oracle_keep_frames
from workloads import random_frame

pytestmark = pytest.mark.gpu


def test_more_frames_than_half_the_compute_units(oracle):
    import paper_2502_00535_amd.binding as nms

    F, n = 129, 4200
    fr = [random_frame(31 + f, n, extent=2500, max_side=90, integer=f % 2 == 0, score_levels=700) for f in range(F)]
    boxes, scores = np.stack([x[0] for x in fr]), np.stack([x[1] for x in fr])
    counts = np.random.default_rng(2).integers(0, n + 1, F).astype(np.int32)
    counts[:4] = [n, 4097, 4096, 0]
    for theta in (0.45, 0.0):   # the second: literal division
        want = oracle_keep_frames(oracle, boxes, scores, np.float32(theta), counts)
        dev = DeviceFrames(nms, boxes, scores, counts)
        assert np.array_equal(dev.fused(theta), want)
        dev.keep.fill_(77)
        nms.nms_run_early_exit_batched(dev.boxes, dev.scores, dev.counts, n, F, theta, dev.keep, dev.run_ws)
        dev.torch.cuda.synchronize()
        assert np.array_equal(dev.keep.cpu().numpy(), want)
