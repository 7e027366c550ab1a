"""Host-only checks of the SpMV layouts beside the row blocks: the plans of the
push, the tile and the one-workgroup layout, executed on the host, give the
plain CSR product exactly on integer data, for even, skewed, empty, long and
mixed rows, every panel count, and row counts around the lanes; a planner or a
relabeling that runs out of memory throws, on whichever thread.  Built from the library's sources; no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_24429_amd", "csrc")


def test_bucket_plans_give_the_csr_product(tmp_path):
    exe = tmp_path / "buckets_check"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread",
                           "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "cpp", "buckets_check.cpp"),
                           os.path.join(CSRC, "host_csr.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    lines = r.stdout.strip().splitlines()
    assert lines[-1] == "done" and len(lines) == 13 * 4 + 8 + 2
    assert lines[-2].startswith("memory ")
    # rows of 4,500 entries among rows of 3 do not fill buckets (the library
    # keeps row blocks there); even rows do
    by = [dict(zip(ln.split()[1::2], ln.split()[2::2])) | {"layout": ln.split()[0]}
          for ln in lines[:-2] if not ln.startswith("small")]
    assert all(d["fragmented"] == "0" for d in by if d["kind"] == "0")
    assert any(d["fragmented"] == "1" for d in by if d["kind"] == "3")
