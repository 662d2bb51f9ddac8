"""Host code of the library on a stand-in HIP runtime (tests/host: every stream a
thread, completion known to the host later than on the device): object
lifetimes, memory accounting, error paths and the choice of solver, without a
GPU. The kernels are stand-ins too, so nothing here is about numbers."""

import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1111_0125_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SOURCES = [os.path.join(CSRC, f) for f in ("capi.cpp", "solver.cpp", "serve.cpp", "tune.cpp")]
SOURCES += [os.path.join(HOST, f) for f in ("hip_stub.cpp", "scenarios.cpp")]


@pytest.fixture(scope="module")
def scenarios(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    out = tmp_path_factory.mktemp("host")
    (out / "align.h").write_text("#define __align__(x) __attribute__((aligned(x)))\n")
    flags = ["-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-include", str(out / "align.h"),
             "-I", os.path.join(ROCM, "include")]

    def compile_one(src):
        obj = str(out / (os.path.basename(src) + ".o"))
        subprocess.run(["g++", *flags, "-c", src, "-o", obj], check=True)
        return obj

    with ThreadPoolExecutor(len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    exe = str(out / "scenarios")
    subprocess.run(["g++", "-o", exe, *objs, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("name", ["lifetime", "launch_error", "small_without_graphs", "small_same_for_blocks",
                                  "budget", "failed_sync", "temporaries", "resident_gives_up",
                                  "resident_together", "resident_launches_are_short", "tuned_sizes",
                                  "bad_links", "groups_on_queues_of_their_own"])
def test_host_scenario(scenarios, name):
    env = {k: v for k, v in os.environ.items() if k != "STAG_TUNE_CACHE"}
    r = subprocess.run([scenarios, name], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stderr
