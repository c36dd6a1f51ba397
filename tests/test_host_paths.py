"""Host paths of libfea.so on the CPU, with the runtime calls it makes played
by the test program (tests/native/host_paths_check.cpp), and host code of its
own (tests/native/mixed_sample_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "native", "host_paths_check.cpp")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(SRC), reason="no g++ or no source")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_paths") / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-rdynamic", SRC,
                    "-o", exe, "-ldl", "-pthread"], check=True)
    return exe


@pytest.mark.parametrize("check", ["waits", "pipe", "header", "bounds", "full", "release"])
def test_host_paths(program, check, tmp_path):
    import paper_1805_03949_amd as fea
    p = subprocess.run([program, fea.LIB_PATH, check, str(tmp_path)], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=120)
    assert p.returncode == 0, p.stdout[-4000:]


def test_sampled_nodes(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(ROOT, "tests", "native", "mixed_sample_check.cpp"), "-o", exe],
                   check=True)
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert p.returncode == 0, p.stdout[-4000:]
