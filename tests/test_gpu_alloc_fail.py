"""`-m gpu`: a batch for which device memory has run out (tests/alloc_fail.cpp, a program of its own whose allocations can be made to
fail)."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_room_for_the_mark_map(tmp_path):
    import paper_2208_05321_amd as pkg
    lib = os.path.dirname(os.path.abspath(pkg.__file__))
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp_path / "alloc_fail")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", f"{rocm}/include",
                           os.path.join(ROOT, "tests", "alloc_fail.cpp"), "-o", exe, "-L", lib, "-lfreqcache", "-L", f"{rocm}/lib", "-lamdhip64", "-ldl",
                           f"-Wl,-rpath,{lib}:{rocm}/lib"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr[-2000:]
