"""The update's memory accesses, checked on the CPU: the classes that the reconstruction kernels apply their update with
(csrc/psd_update.h) compiled for the host under the address sanitizer (tests/host/update_check.cpp)."""
import os
import subprocess

from paper_1512_06216_amd import build
from tests.conftest import ROOT


def test_update_touches_no_element_of_another_tile_and_nothing_past_the_end(tmp_path):
    clang = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "lib", "llvm", "bin", "clang++")
    exe = str(tmp_path / "update_check")
    subprocess.run([clang, "-x", "c++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "include"), "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "host", "update_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith("all right\n"), r.stdout[-3000:]
