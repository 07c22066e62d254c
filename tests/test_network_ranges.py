"""Range check of the proposal network's launches (CPU): the policy runtime's host code is
compiled under AddressSanitizer and UndefinedBehaviorSanitizer against a stand-in HIP runtime
and launchers (tests/networkcheck) that check every range which the pass over the network, the
weight gradients, the parameter pass, the loss and the head read or write: inside its buffer,
apart from what the same launch and the call's other launches use, and written before it is
read.  Planted faults (a buffer registered too short, a launch whose results are taken
as not written) show that each of them is seen."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CS = os.path.join(ROOT, "paper_2409_10469_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ is not available")
    exe = str(tmp_path_factory.mktemp("network") / "networkcheck")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-Wall", "-Wno-unknown-pragmas", "-Werror", "-I", os.path.join(ROOT, "tests", "hostcheck"),
           "-I", os.path.join(ROOT, "include"), "-I", CS, os.path.join(ROOT, "tests", "networkcheck", "network.cpp"),
           os.path.join(CS, "mppi_policy.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def _run(exe, *args):
    return subprocess.run([exe, *args], capture_output=True, text=True, timeout=300)


def test_network_launches_stay_in_range(exe):
    r = _run(exe)
    assert r.returncode == 0, (r.stdout[-4000:], r.stderr[-4000:])
    assert "faults: 0" in r.stdout
    assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr


@pytest.mark.parametrize("plant", ["short-input", "short-target", "short-output", "short-indexed-input",
                                   "short-indexed-target", "short-indices", "short-gradient", "short-parameters",
                                   "short-loss", "short-workspace", "short-centre", "short-std", "short-state",
                                   "short-command", "unwritten-network", "unwritten-gradients", "unwritten-copies"])
def test_planted_faults_are_seen(exe, plant):
    r = _run(exe, plant)
    assert r.returncode == 1 and "faults: 0" not in r.stdout, (plant, r.stdout[-2000:], r.stderr[-2000:])
