"""How attention is split over workgroups and wavefronts (csrc/attn_split.h, on the CPU): work lists of many batches hold
every key once and fit what holds them, and the rules choose what they were measured to choose."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")


def test_attention_split(tmp_path):
    exe = str(tmp_path / "attn_split")
    r = subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(NATIVE, "one_workgroup"), "-I", os.path.join(ROOT, "paper_2503_05931_amd", "csrc"),
                        os.path.join(NATIVE, "attn_split.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
