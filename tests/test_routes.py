"""The launches, copies and allocations that calls of the library make, on a stand-in for the HIP
runtime (tests/routes_check.cpp, linked with the built library; no GPU needed)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2110_14934_amd")


@pytest.fixture(scope="session")
def exe(tmp_path_factory):
    cxx = shutil.which("g++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if cxx is None or not os.path.exists(os.path.join(rocm, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    if not os.path.exists(os.path.join(LIB, "libgmm.so")):
        pytest.skip("the library is not built")
    out = str(tmp_path_factory.mktemp("routes") / "routes_check")
    cmd = [cxx, "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
           f"-I{os.path.join(ROOT, 'include')}", os.path.join(HERE, "routes_check.cpp"), f"-L{LIB}", "-l:libgmm.so",
           f"-Wl,-rpath,{LIB}", f"-Wl,-rpath,{rocm}/lib", f"-L{rocm}/lib", "-Wl,--allow-shlib-undefined", "-pthread", "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    return out


@pytest.mark.parametrize("check", ["gap", "coherence", "overlap", "detach", "round_trip", "exec_tuning", "residency",
                                   "cache_policy", "state_io", "autotune", "staging"])
def test_routes(exe, check):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "routes ok" in r.stdout, r.stdout + r.stderr
