"""The solver engine and the C ABI's drivers on the host (csrc/hub_engine.hip,
csrc/hub_api.hip), without a GPU.

tests/engine_host.cpp plays the device (launches take effect at once, with numbers of its
own) and leads the engine into states that a device at work reaches only now and then.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1804_07195_amd", "csrc")
ROCM = "/opt/rocm/include"
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "hip")),
                                reason="no host compiler or no HIP headers")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("engine") / "engine_host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))",
                    "-DHIP_SYMBOL(x)=(&x)", "-I" + ROCM, "-I" + os.path.join(ROOT, "include"),
                    "-I" + CSRC, "-x", "c++", os.path.join(CSRC, "hub_engine.hip"), os.path.join(CSRC, "hub_api.hip"),
                    os.path.join(ROOT, "tests", "engine_host.cpp"), "-lpthread", "-o", out], check=True)
    return out


@pytest.mark.parametrize("scenario", ["lost_publication", "refusal_keeps_cache", "tables_of_fields",
                                      "gang_without_an_answer", "gangs_that_never_meet", "kernels_by_request",
                                      "turns", "cus_of_the_stream", "like_with_like"])
def test_engine(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
