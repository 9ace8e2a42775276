"""The workloads by which this library's speed is judged: what a user has it do, through its public
entry points, over the sizes that detectors emit.

Scenes are made on the GPU from the seed alone, with the distributions of this repository's synthetic
workloads: objects with sixteen jittered candidates each ("clusters"), a dense crowd with tied scores
("crowd"), regressed pyramid anchors of which two in a hundred score high ("anchors").
"""
import math

import torch

from paper_2502_00535_amd import binding as nms

DEVICE = "cuda:0"

# What a detector's post-processing commonly asks of the variants call: the sequential rule on
# intersection over union, strictly above the threshold, continuous coordinates.
DETECTOR = {"rule": "greedy", "measure": "iou", "compare": "gt", "pixel_offset": 0.0}


def _case(name, call, scene, frames, n, theta, ragged=False, labels=0):
    c = {"call": call, "scene": scene, "frames": frames, "n": n, "theta": theta, "ragged": ragged, "labels": labels}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one 1080p video frame with few detections: nothing but the cost of a call
        _case("frame_360", "frame", "clusters", 1, 360, 0.5),
        # one 1080p frame, the capacity at which single-frame latency is quoted
        _case("frame_1024", "frame", "clusters", 1, 1024, 0.5),
        # one 4K frame at the paper's full capacity
        _case("frame_4096", "frame", "clusters", 1, 4096, 0.5),
        # one 4K picture of a dense crowd, with exact score ties
        _case("crowd_16384", "frame", "crowd", 1, 16384, 0.3),
        # sixty-four cameras, a step of the serving loop on buffers that stay (a plan made once)
        _case("stream_64x1024", "plan", "clusters", 64, 1024, 0.5),
        # a batch of pictures with different numbers of detections, an odd capacity
        _case("ragged_48x1777", "batch", "clusters", 48, 1777, 0.5, ragged=True),
        # a throughput batch of single-shot detector outputs, the automatic route
        _case("anchors_256x4096", "batch", "anchors", 256, 4096, 0.45),
        # the same batch where the caller wants every pair evaluated (a running time that the data does not change)
        _case("all_pairs_256x4096", "all_pairs", "anchors", 256, 4096, 0.45),
        # the three steps one by one, for a caller that uses the order and the elimination mask itself
        _case("steps_16x4096", "steps", "clusters", 16, 4096, 0.5),
        # the sequential rule on a small batch of odd size
        _case("greedy_24x3000", "greedy", "anchors", 24, 3000, 0.45),
        # one picture through an IoU detector's post-processing
        _case("detector_frame_4096", "detector", "clusters", 1, 4096, 0.5),
        # a ragged batch of multi-class detections, per-class suppression
        _case("detector_128x3000_classes", "detector", "anchors", 128, 3000, 0.6, ragged=True, labels=20),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["frame", "frame", "plan", "batch", "batch", "batch", "all_pairs", "steps", "greedy", "detector",
                       "detector", "paper_iou"])
    # boxes per frame: the mask of the steps and of the sequential rule grows with the square
    n_hi = {"frame": 32768, "batch": 16384, "all_pairs": 16384, "plan": 4096}.get(call, 8192)
    n = _log_uniform(rng, 64, n_hi)
    slots = 2 ** 32 if call in ("frame", "plan", "batch", "all_pairs") else 2 ** 30
    frames = 1 if call == "frame" else _log_uniform(rng, 1, max(1, min(512, slots // (n * n))))
    scene = rng.choice(["clusters", "crowd"] if n > 4096 else ["clusters", "anchors"])
    theta = rng.choice([0.3, 0.4, 0.45, 0.5, 0.6, 0.7])
    ragged = call != "frame" and call != "plan" and rng.random() < 0.4
    labels = rng.choice([0, 5, 20]) if call in ("detector", "paper_iou") else 0
    return _case(None, call, scene, frames, n, theta, ragged, labels)


# ---------------------------------------------------------------- scenes

def _beta(gen, a, b, shape):
    """Beta(a, b) for whole a and b: the a-th smallest of a + b - 1 uniform numbers."""
    u = torch.rand((*shape, a + b - 1), generator=gen, device=DEVICE)
    return u.kthvalue(a, dim=-1).values


def _boxes(cx, cy, w, h, width, height):
    """Corner form, clipped to the picture, at least one pixel wide and high."""
    x1 = (cx - 0.5 * w).clamp(0.0, width - 2.0)
    y1 = (cy - 0.5 * h).clamp(0.0, height - 2.0)
    x2 = torch.maximum((cx + 0.5 * w).clamp(0.0, width - 1.0), x1 + 1.0)
    y2 = torch.maximum((cy + 0.5 * h).clamp(0.0, height - 1.0), y1 + 1.0)
    return torch.stack([x1, y1, x2, y2], dim=-1)


def _candidates(gen, f, n, objects, cx, cy, size, rho):
    """n candidates per frame, each of one of the frame's objects: centre noise 8 % of the side,
    sides scaled by exp(N(0, 0.1)), in random order."""
    pick = torch.rand((f, n), generator=gen, device=DEVICE).argsort(dim=1) % objects

    def normal():
        return torch.randn((f, n), generator=gen, device=DEVICE)
    w = (size * rho.sqrt()).gather(1, pick)
    h = (size / rho.sqrt()).gather(1, pick)
    x = cx.gather(1, pick) + normal() * 0.08 * w
    y = cy.gather(1, pick) + normal() * 0.08 * h
    return x, y, w * (0.1 * normal()).exp(), h * (0.1 * normal()).exp()


def _clusters(gen, f, n):
    """Objects anywhere in the picture, sixteen candidates each; 1080p up to some 2000 boxes, else 4K."""
    width, height, lo, hi = (1920.0, 1080.0, 32.0, 256.0) if n <= 2048 else (3840.0, 2160.0, 24.0, 384.0)
    m = max(1, n // 16)

    def uniform(a, b):
        return a + (b - a) * torch.rand((f, m), generator=gen, device=DEVICE)
    x, y, w, h = _candidates(gen, f, n, m, uniform(0.0, width), uniform(0.0, height), uniform(lo, hi),
                             torch.exp2(uniform(-1.0, 1.0)))
    return _boxes(x, y, w, h, width, height), _beta(gen, 5, 2, (f, n))


def _crowd(gen, f, n):
    """Near-square objects on a jittered lattice, neighbours overlapping; one score in a hundred tied."""
    width, height = 3840.0, 2160.0
    g = max(2, int(round(math.sqrt(n / 16.0))))
    m = g * g
    cell = torch.arange(m, device=DEVICE).expand(f, m)

    def uniform(a, b):
        return a + (b - a) * torch.rand((f, m), generator=gen, device=DEVICE)
    cx = ((cell % g) + 0.5 + uniform(-0.5, 0.5)) * (width / g)
    cy = (torch.div(cell, g, rounding_mode="floor") + 0.5 + uniform(-0.5, 0.5)) * (height / g)
    x, y, w, h = _candidates(gen, f, n, m, cx, cy, uniform(24.0, 96.0), torch.exp2(uniform(-0.1, 0.1)))
    scores = _beta(gen, 5, 2, (f, n))
    tied = torch.rand((f, n), generator=gen, device=DEVICE) < 0.01
    other = torch.randint(0, n, (f, n), generator=gen, device=DEVICE)
    scores = torch.where(tied, scores.gather(1, other), scores)
    return _boxes(x, y, w, h, width, height), scores


def _anchors(gen, f, n):
    """Anchors of a six-level pyramid on a 512 x 512 picture, drawn without replacement, regressed."""
    rows = []
    for stride in (8, 16, 32, 64, 128, 256):
        centre = (torch.arange(512 // stride, device=DEVICE) + 0.5) * stride
        gy, gx = torch.meshgrid(centre, centre, indexing="ij")
        for aspect in (0.5, 1.0, 2.0):
            side = torch.full_like(gx, 4.0 * stride)
            rows.append(torch.stack([gx, gy, side * math.sqrt(aspect), side / math.sqrt(aspect)], -1).reshape(-1, 4))
    table = torch.cat(rows)
    pick = torch.rand((f, table.shape[0]), generator=gen, device=DEVICE).argsort(dim=1)[:, :n]
    a = table[pick]

    def normal():
        return torch.randn((f, n), generator=gen, device=DEVICE)
    x = a[..., 0] + 0.1 * normal() * a[..., 2]
    y = a[..., 1] + 0.1 * normal() * a[..., 3]
    boxes = _boxes(x, y, a[..., 2] * (0.1 * normal()).exp(), a[..., 3] * (0.1 * normal()).exp(), 512.0, 512.0)
    hot = torch.rand((f, n), generator=gen, device=DEVICE) < 0.02
    return boxes, torch.where(hot, _beta(gen, 8, 2, (f, n)), _beta(gen, 1, 8, (f, n)))


_SCENES = {"clusters": _clusters, "crowd": _crowd, "anchors": _anchors}


# ---------------------------------------------------------------- a case's state, one pass, its work

def prepare(case, seed):
    f, n, call = case["frames"], case["n"], case["call"]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    boxes, scores = _SCENES[case["scene"]](gen, f, n)
    s = {"case": case, "boxes": boxes.float().contiguous(), "scores": scores.float().contiguous(), "counts": None,
         "classes": None, "keep": torch.empty((f, n), dtype=torch.uint8, device=DEVICE)}
    if case["ragged"]:  # between half full and full
        s["counts"] = torch.randint(n // 2, n + 1, (f,), generator=gen, device=DEVICE, dtype=torch.int32)
    if case["labels"]:
        s["classes"] = torch.randint(0, case["labels"], (f, n), generator=gen, device=DEVICE, dtype=torch.int32)
    size = {"greedy": nms.nms_greedy_workspace_bytes, "detector": nms.nms_ex_workspace_bytes,
            "paper_iou": nms.nms_ex_workspace_bytes, "steps": nms.nms_sort_workspace_bytes}.get(call, nms.nms_workspace_bytes)
    s["workspace"] = torch.empty(max(256, size(n, f)), dtype=torch.uint8, device=DEVICE)
    if call == "steps":
        # the step that fills the mask writes its lower triangle only
        s["order"] = torch.zeros((f, n), dtype=torch.int32, device=DEVICE)
        s["sorted5"] = torch.empty((f, 5 * nms.nms_padded_n(n)), dtype=torch.float32, device=DEVICE)
        s["mask"] = torch.zeros((f, nms.nms_mask_words(n)), dtype=torch.int64, device=DEVICE)
    if call == "plan":
        s["plan"] = nms.RunPlan(s["boxes"], s["scores"], s["counts"], n, f, case["theta"], s["keep"], s["workspace"])
    return s


def run(s):
    c = s["case"]
    f, n, theta, call = c["frames"], c["n"], c["theta"], c["call"]
    boxes, scores, counts, keep, ws = s["boxes"], s["scores"], s["counts"], s["keep"], s["workspace"]
    if call == "frame":
        nms.nms_run_ws(boxes, scores, n, theta, keep, ws)
    elif call == "plan":
        s["plan"]()
    elif call == "batch":
        nms.nms_run_batched(boxes, scores, counts, n, f, theta, keep, ws)
    elif call == "all_pairs":
        nms.nms_run_ranked_batched(boxes, scores, counts, n, f, theta, keep, ws)
    elif call == "steps":
        nms.nms_sort_batched(boxes, scores, counts, n, f, s["order"], s["sorted5"], ws)
        nms.nms_overlap_mask_batched(s["sorted5"], counts, n, f, theta, s["mask"])
        nms.nms_reduce_batched(s["mask"], s["order"], counts, n, f, keep)
        return {"keep": keep, "order": s["order"], "sorted5": s["sorted5"], "mask": s["mask"]}
    elif call == "greedy":
        nms.nms_run_greedy_batched(boxes, scores, counts, n, f, theta, keep, ws)
    elif call == "detector":
        nms.nms_run_ex_batched(boxes, scores, counts, n, f, theta, keep, ws, classes=s["classes"], **DETECTOR)
    elif call == "paper_iou":
        nms.nms_run_ex_batched(boxes, scores, counts, n, f, theta, keep, ws, measure="iou", classes=s["classes"])
    else:
        raise ValueError(call)
    return keep


def work(case):
    """Each input read and each output written once.  One pair test is 13 operations (Algorithm 1:
    two extents of min, max, subtract, add and floor, a product, a division, a compare).  Calls that
    promise every pair count them all; the others cannot do without one test per box."""
    f, n = case["frames"], case["n"]
    boxes = f * n
    moved = boxes * (16 + 4 + 1)
    if case["ragged"]:
        boxes = 0.75 * boxes  # counts are uniform between half and full
        moved = boxes * (16 + 4) + f * (n + 4)
    moved += 4 * boxes if case["labels"] else 0
    tests = boxes
    if case["call"] in ("all_pairs", "steps"):
        tests = 0.5 * boxes * (boxes / f - 1)
    if case["call"] == "steps":
        pad = (n + 63) // 64 * 64
        # order, box table and mask triangle are outputs, and the next step's inputs
        moved += 2 * (4 * boxes + 20 * f * pad + 8 * f * (pad // 64) * (pad + 64) / 2)
    return {"bytes": float(moved), "flops": 13.0 * float(tests)}


def tolerance(case):
    """Keep bytes, order and mask are whole numbers and the box table holds copies and areas whose
    every operation is rounded on its own in a stated order: one result is correct."""
    return "exact"
