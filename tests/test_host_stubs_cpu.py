"""The library's host code over a HIP runtime that only takes notes
(host_stubs.cpp): the streams it uses and the order of its launches and waits, which
one GPU cannot show."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_08063_amd", "csrc")


def _build(out, flags=()):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    subprocess.run([gxx, "-O1", "-g", "-std=c++17", *flags, "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host_stubs.cpp"),
                    os.path.join(CSRC, "fwi_runtime.cpp"), os.path.join(CSRC, "revolve.cpp"),
                    "-pthread", "-o", out], check=True)
    return out


@pytest.fixture(scope="module")
def stubs(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("stubs") / "stubs"))


def _run(exe, *args):
    p = subprocess.run([exe, *args], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
    return p.stdout.split("\n")[:-1]


def test_side_streams_only_on_the_callers_device(stubs):
    """Launch groups of one advance go to side streams, but not where the caller's
    stream belongs to another device than the current one: side streams are of the
    current device."""
    steps, streams = _run(stubs, "lanes", "0")[0].split()[1:4:2]
    assert int(steps) == 8 and int(streams) == 2
    assert _run(stubs, "lanes", "1") == ["steps 8 streams 1 caller 1"]


def test_a_created_job_has_nothing_in_flight(stubs):
    """fwi_job_create synchronises its stream after all it enqueues: the job may be
    advanced on another stream, whose first step reads the cleared levels."""
    did = _run(stubs, "create")
    assert did[0] == "check" and {"tables", "kappa", "frames", "fill"} <= set(did)
    assert did[-1] == "sync"


@pytest.mark.parametrize("order,shots,kind", [
    (4, 1, "tile"), (4, 6, "tile"), (4, 8, "tile"), (4, 16, "tile"), (4, 32, "marching"),
    (8, 1, "tile"), (8, 6, "tile"), (8, 8, "marching"), (8, 32, "marching")])
def test_two_step_marching_by_cells_and_order(order, shots, kind, stubs):
    """Forward launches of 2.5 M cells and more march two steps at 8th order, of 10 M
    and more at 4th order."""
    assert _run(stubs, "forward", str(order), str(shots)) == [kind + " steps"]
