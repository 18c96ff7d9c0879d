"""The library's host runtime on a stand-in HIP runtime (no device):
tests/hip_stub/host_path.cpp defines the HIP functions that libhwr calls, runs
a scenario through the C ABI and checks what the library asked of them."""
import os
import shutil
import subprocess

import pytest

from paper_2608_14575_amd import hwr

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.dirname(hwr.LIB_PATH)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    if not os.path.exists(hwr.LIB_PATH):
        from paper_2608_14575_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("hip_stub") / "host_path")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__",
                    "-isystem", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "hip_stub", "host_path.cpp"), f"-L{PKG}", "-lhwr", f"-Wl,-rpath,{PKG}",
                    f"-Wl,-rpath-link,{os.path.join(ROCM, 'lib')}", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["memory_short", "growing_batches", "few_compute_units",
                                      "upload_beside_the_stream", "chunk_path_instead"])
def test_host_runtime(driver, scenario):
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
