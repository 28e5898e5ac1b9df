"""Tables that the tensors of a group share (csrc/excp_device.h), in a small program of their own; no GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rows_and_cells_have_places_of_their_own(tmp_path):
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))))
    exe = str(tmp_path / "host_tables_check")
    subprocess.run([os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    "-fsanitize=address,undefined", os.path.join(ROOT, "tests", "host_tables_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
