"""The rank step by counting (batches of up to 32,768 boxes) against the radix sort that larger
batches take, through nms_sort_batched: the order and the whole box table, bit for bit."""
import numpy as np
import pytest

from workloads import random_frame, scores_of_every_kind

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nms():
    import torch

    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2502_00535_amd.binding as binding

    return binding


def rank(nms, boxes, scores, counts):
    import torch

    dev = torch.device("cuda:0")
    frames, n = scores.shape
    order = torch.full((frames, n), -7, dtype=torch.int32, device=dev)
    table = torch.full((frames, 5 * nms.nms_padded_n(n)), 7.0, dtype=torch.float32, device=dev)
    ws = torch.empty(max(256, nms.nms_sort_workspace_bytes(n, frames)), dtype=torch.uint8, device=dev)
    c = None if counts is None else torch.from_numpy(counts).to(dev)
    nms.nms_sort_batched(torch.from_numpy(boxes).to(dev), torch.from_numpy(scores).to(dev), c, n, frames, order, table, ws)
    torch.cuda.synchronize()
    return order.cpu().numpy(), table.cpu().numpy()


def oracle_rank(boxes, scores, n_pad):
    """Order and box table of one frame, from a stable sort on the host."""
    c = len(scores)
    order = np.argsort(-scores.astype(np.float64), kind="stable")
    rows = np.zeros((n_pad, 4), np.float32)
    rows[:c] = boxes[order]
    one = np.float32(1)
    areas = ((rows[:, 2] - rows[:, 0]) + one) * ((rows[:, 3] - rows[:, 1]) + one)
    return order, np.concatenate([rows.reshape(-1), areas])


# The small batch counts, with 16 or 64 elements per workgroup (both occur below; the last that counts has 32,768
# boxes), the large one sorts.
@pytest.mark.parametrize("n,few", [(1, 1), (63, 1), (64, 300), (65, 1), (129, 130), (384, 1), (385, 1), (1000, 4), (1000, 17), (1000, 32),
                                   (1025, 3), (2048, 4), (2048, 16), (4095, 1), (4095, 4), (4096, 1), (4096, 2), (4096, 5), (4096, 8)])
def test_counted_ranks_equal_sorted_ranks(nms, n, few):
    print(f"case n={n} frames={few}", flush=True)
    many = max(few, 32768 // n + 1)  # a batch that sorts
    assert n * few <= 32768 < n * many  # the bound that test_host_logic.py pins
    rng = np.random.default_rng(n + few)
    boxes = np.zeros((many, n, 4), np.float32)
    scores = np.zeros((many, n), np.float32)
    distinct = [random_frame(100 * n + f, n, extent=500, max_side=90, integer=f % 2 == 0, score_levels=(0, 5, 1)[f % 3])
                for f in range(3)]
    for f in range(many):
        boxes[f], scores[f] = distinct[f % 3]
    for f in range(0, few, 4):
        scores[f] = np.resize(scores_of_every_kind(n, n + f), n)
    for counts in (None, rng.integers(-1, n + 2, many).astype(np.int32)):
        if counts is not None:
            counts[0], counts[few - 1] = n - 1, n // 2
        want_order, want_table = rank(nms, boxes, scores, counts)
        order, table = rank(nms, boxes[:few], scores[:few], None if counts is None else counts[:few])
        assert np.array_equal(order, want_order[:few])
        assert np.array_equal(table.view(np.uint32), want_table[:few].view(np.uint32))
        for f in range(few):
            c = n if counts is None else int(np.clip(counts[f], 0, n))
            host_order, host_table = oracle_rank(boxes[f, :c], scores[f, :c], nms.nms_padded_n(n))
            assert np.array_equal(order[f, :c], host_order), f"frame {f}"
            assert np.array_equal(table[f].view(np.uint32), host_table.view(np.uint32)), f"frame {f}"
