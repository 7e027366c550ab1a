"""The library's host paths against a stand-in for the HIP runtime (device
memory is host memory, kernels do nothing; tests/cpp/fake_device_check.cpp):
every device allocation of a user's calls fails in turn, and no call leaves
memory behind, leaves things half done or fails for want of a bucketed layout;
products with the loaded values launch nothing for layouts they don't use.  No
GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_out_of_memory_paths(tmp_path):
    from paper_2510_24429_amd import _lib
    _lib.lib()
    exe = tmp_path / "fake_device_check"
    # (-rdynamic: the stand-in's functions come before the runtime's)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-rdynamic", "-pthread",
                           "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", "cpp", "fake_device_check.cpp"),
                           "-o", str(exe), "-ldl"])
    r = subprocess.run([str(exe), os.path.join(ROOT, "paper_2510_24429_amd", "libpdhg.so")],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    lines = r.stdout.strip().splitlines()
    assert lines[-1] == "done" and len(lines) == 7 + 4 + 1 + 1 + 1
