"""Kernel arguments that come in a tail (csrc/kernel_tail.h, on the CPU): offsets and lengths follow from the kernel's type and the
list of arguments, and a tail is read wherever a kernel's leading arguments end (no alignment is promised that is not there)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")


def test_kernel_tail(tmp_path):
    exe = str(tmp_path / "kernel_tail")
    r = subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(NATIVE, "one_workgroup"), "-I", os.path.join(ROOT, "paper_2503_05931_amd", "csrc"),
                        os.path.join(NATIVE, "kernel_tail.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
