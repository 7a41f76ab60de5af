"""One wave clears the records or counters for all of its launch: every wait for it ends, and nothing is lost, in whatever
order the workgroups of two launches that fill the chip start."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("clear_once") / "model")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-I", os.path.join(HERE, "..", "paper_2311_05782_amd", "csrc"),
                    os.path.join(HERE, "clear_once_model.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("order", ["ascending", "descending", "random"])
@pytest.mark.parametrize("slots", [1, 2, 4])
def test_whatever_order_the_workgroups_start_in(model, order, slots):
    r = subprocess.run([model, order, str(slots)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    assert r.returncode == 0, r.stdout
