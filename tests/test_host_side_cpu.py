"""-m "not gpu": the host side of libdba on a stand-in for the HIP runtime, whose GPU runs when the scenario says so."""
import os
import shutil
import subprocess

import pytest

from paper_1804_06609_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("host_side") / "host_side_driver")
    build = subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-Wall", "-rdynamic", os.path.join(HERE, "host_side_driver.cpp"), "-o", exe, "-ldl"],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr
    return exe


@pytest.mark.parametrize("scenario", ["launch_errors", "calls_of_a_step", "steps_under_way", "places_made_empty"])
def test_host_side(driver, scenario):
    run = subprocess.run([driver, binding.LIB_PATH, scenario], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == scenario + " ok\n", run.stdout + run.stderr
