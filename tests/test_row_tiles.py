"""The addresses of a 16-row tile's loads (CPU): csrc/gemm_common.h compiled for the host, with a buffer load that returns
the address it would read, for rows up to the widest of which a descriptor's offsets reach 16; products over wider ones take
other tiles."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native", "one_workgroup")


def test_row_tiles_of_any_width(tmp_path):
    exe = str(tmp_path / "frag_rows")
    r = subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-w", "-I", NATIVE,
                        "-I", os.path.join(ROOT, "paper_2503_05931_amd", "csrc"),
                        os.path.join(NATIVE, "frag_rows.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
