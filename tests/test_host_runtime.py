"""Host code of the library against a stand-in for the HIP runtime (CPU only).

tests/host_runtime.c defines the runtime's functions itself and is linked to the
built library, so the launches, allocations, waits and attributes that the host
code asks for can be counted and the event times of the autotuner scripted:

* depth of the regular-voxel march: a depth that is ahead by less than the noise
  of the timings does not replace the default, nor does one disturbed timing
  decide; a depth that pays is taken and kept for the grid; after a failed
  timing the default stays and the next problem times again;
* dynamic LDS: on each of two devices of one process, every launch with more
  than 64 KB follows the attribute that allows it on that device;
* setup: no more allocations, frees and waits than 49, 13 and 8 (those of the
  library before the lists of cut elements were built at setup), and everything
  freed with the problem.
"""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gcc = shutil.which("gcc")
    if not gcc:
        pytest.skip("gcc not found")
    from paper_2601_02172_amd import xfft, build
    xfft._lib()                                  # the library is built and loads
    exe = str(tmp_path_factory.mktemp("host_runtime") / "host_runtime")
    pkg = os.path.dirname(build.LIB)
    r = subprocess.run([gcc, "-O1", "-g", "-std=gnu11", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host_runtime.c"), "-o", exe, "-L", pkg, "-lxfft",
                        f"-Wl,-rpath,{pkg}", "-Wl,--allow-shlib-undefined"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def _run(exe, *args):
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout + r.stderr)
    assert "checks passed" in r.stdout


@pytest.mark.parametrize("case", ["close", "outlier", "faster", "failed"])
def test_depth_of_the_regular_march(program, case):
    _run(program, "depth", case)


@pytest.mark.parametrize("n,precision", [(128, 0), (96, 1), (108, 0)])
def test_lds_attribute_on_every_device(program, n, precision):
    _run(program, "devices", str(n), str(precision))


@pytest.mark.parametrize("n0,n1", [(16, 16), (24, 18)])
def test_calls_of_a_setup(program, n0, n1):
    _run(program, "setup", str(n0), str(n1), "49", "13", "8")
