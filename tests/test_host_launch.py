"""The host side of tuning and launches on the CPU, with a stand-in for the
device runtime whose kernel costs and failures the test sets
(tests/native/host_device.cpp, tests/host_launch.py)."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def device(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    from paper_2412_17543_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2412_17543_amd.build import build
        build()
    out = str(tmp_path_factory.mktemp("device") / "host_device.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "native", "host_device.cpp"),
                    "-o", out], check=True, capture_output=True)
    return out


def _run(device, *args):
    r = subprocess.run([sys.executable, os.path.join(HERE, "host_launch.py"), device] + [str(a) for a in args],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr


@pytest.mark.parametrize("schur,neumann", [
    (8, 16),          # a quarter and a half of the blocks of one per compute unit (few segments, cheap sums)
    (64, 300),        # whole numbers of blocks a compute unit
    (24, 48),
])
def test_tuned_configuration_can_be_pinned(device, schur, neumann):
    _run(device, "pinned", schur, neumann)


@pytest.mark.parametrize("schur,interior", [(8, 232), (24, 232)])
def test_interior_product_tuned_on_its_own_splits(device, schur, interior):
    _run(device, "interior", schur, interior)


@pytest.mark.parametrize("cfg", [(2, 1, 5, 2), (2, 1, 4, 3)])       # waves, tiles in flight
def test_refused_launch_configuration_changes_nothing(device, cfg):
    _run(device, "refused", *cfg)


@pytest.mark.parametrize("cfg", [(8, 0, 8, 4), (2, 1, 4, 2)])
def test_failed_launch_configuration_changes_nothing(device, cfg):
    _run(device, "failed", *cfg)
