"""The protocols by which the kernels' waves and blocks share words
(csrc/acs_protocol.hpp), run on the CPU from the header that the kernels
include: the result may not depend on which wave is late, nor on what earlier
launches left in the words, and all blocks of a launch whose blocks wait for each
other have to be resident."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1605_02669_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("protocol") / "driver")
    res = subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                          "-I", CSRC, os.path.join(HERE, "protocol_driver.cpp"), "-o", exe,
                          "-lpthread"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


@pytest.mark.parametrize("name", ["queue_round", "barrier", "sync_residency",
                                  "seq_groups"])
def test_protocol(driver, name):
    r = subprocess.run([driver, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
