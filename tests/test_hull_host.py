"""The pair test is monotone in the victim's box: a hull around several victims is eliminated where one of them is, whatever the
rounding (coordinates of very different sizes, thresholds at both ends of the division-free range, boxes that just touch).  What the kernels
in order of place rest on, tiles of outranking boxes with their hull and least T, is in test_place_host.py."""
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_hull_never_loses_an_elimination(tmp_path):
    exe = tmp_path / "hull_driver"
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    os.path.join(ROOT, "tests", "host", "hull_driver.cpp"), "-o", str(exe)], check=True)
    rng = np.random.default_rng(1)
    lines = []
    for _ in range(20000):
        scale = np.float32(2.0 ** rng.integers(-10, 30))
        size = np.float32(2.0 ** rng.integers(-6, 8))
        grid = rng.random() < 0.5

        def box(centre, spread):
            p = centre + rng.normal(0, spread, 2)
            wh = np.abs(rng.normal(0, size, 2))
            if grid:
                p, wh = np.round(p), np.round(wh)
            return np.concatenate([p, p + wh]).astype(np.float32)
        centre = rng.normal(0, scale, 2)
        c = box(centre, 0)
        k = int(rng.integers(1, 5))
        victims = [c if rng.random() < 0.2 else box(centre, size / 2) for _ in range(k)]
        theta = np.float32(rng.choice([0.3, 0.45, 0.5, 0.7, 1.0, 2.0 ** -40, 0.01, 1.3]))
        lines.append(" ".join(repr(float(x)) for x in (theta, *c)) + f" {k}")
        lines += [" ".join(repr(float(x)) for x in v) for v in victims]
    out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split()
    assert int(out[1]) == 0 and int(out[3]) > 5000, out
