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
