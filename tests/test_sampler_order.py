"""The workgroup that ends a step -- a greedy one: sampler and embedding of what is fed next; a plain one: argmax -- with
its wavefronts in any order (CPU): the kernels' own source, compiled for the host with one fiber per thread."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native", "one_workgroup")


def test_sampler_does_not_depend_on_the_order_of_wavefronts(tmp_path):
    exe = str(tmp_path / "sampler")
    r = subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-w", "-I", NATIVE,
                        "-I", os.path.join(ROOT, "paper_2503_05931_amd", "csrc"),
                        os.path.join(NATIVE, "sampler.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
