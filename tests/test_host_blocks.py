"""The pool of pinned host blocks when calls fail, and calls that run out of host
memory (tests/c/pool_test.cpp: the built libmpt.so on the CPU, with stand-ins for
the HIP calls it makes)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_failing_calls_keep_the_blocks(tmp_path):
    exe, lib = str(tmp_path / "pool_test"), os.path.join(ROOT, "paper_2609_13692_amd")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-isystem",
                           "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           os.path.join(HERE, "c", "pool_test.cpp"), "-o", exe, "-L", lib, "-lmpt",
                           "-L", "/opt/rocm/lib", "-lamdhip64", f"-Wl,-rpath,{lib}:/opt/rocm/lib"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks hold" in r.stdout, r.stdout + r.stderr
