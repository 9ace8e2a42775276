"""What the kernels in order of place leave out, on the CPU, from the header that the kernels include."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = tmp_path_factory.mktemp("host") / "place_driver"
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    os.path.join(ROOT, "tests", "host", "place_driver.cpp"), "-o", str(exe)], check=True)
    return str(exe)


def test_no_tile_behind_the_last_is_reached(driver):
    """An infinite box, or one whose area overflows, reaches every T, infinity included: lanes that stand for no tile
    have to be left out by their number (rows behind the table, and words behind a row's place, were read and written)."""
    out = subprocess.run([driver, "reach"], capture_output=True, text=True, check=True).stdout.split()
    assert int(out[1]) > 100000 and int(out[3]) == 0, out


def test_labels_are_told_apart_and_spread(driver):
    """Bin and bits 4 to 7 name a label from 0 to 255; sixteen labels in steps of 1, 16 or 17 take more than half of the bins
    between them where the steps allow it (one bin for all is a grid without classes)."""
    out = subprocess.run([driver, "bins"], capture_output=True, text=True, check=True).stdout.split("\n")
    bins = {int(a): int(b) for a, b in (line.split() for line in out if line)}
    assert all(0 <= b < 16 for b in bins.values())
    assert len({(bins[n], n & 0xf0) for n in range(256)}) == 256
    assert len({bins[n] for n in range(16)}) == 16 and len({bins[16 * n] for n in range(16)}) == 16
    assert len({bins[20 * n] for n in range(16)}) > 8


def test_no_eliminator_lies_in_a_tile_that_does_not_reach_the_victim(driver):
    """The hull, the least T and the reach predicate of the kernels against the definition (float32, IEEE division), both measures, both
    compares, pixel offsets 1 and 0, boxes without area, tiles that are not full, thresholds at both ends of the division-free range,
    coordinates of very different sizes, boxes that just touch."""
    out = subprocess.run([driver, "tiles"], capture_output=True, text=True, check=True).stdout.strip().split("\n")
    assert len(out) == 6
    for line in out:
        form, violations, hits, reached, asked = line.split()
        assert int(violations) == 0 and int(hits) > 50000 and 5000 < int(asked) - int(reached), line
