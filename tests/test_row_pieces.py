"""Addresses and entries of the 16-byte pieces that ballot rows are read in,
compiled for the CPU (tests/row_pieces.cpp): every size up to several pieces at
every alignment, arrays of less than one piece among them."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_row_pieces(tmp_path):
    exe = str(tmp_path / "row_pieces")
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "row_pieces.cpp"), "-o", exe], check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.stdout.strip() == "ok" and run.returncode == 0, run.stdout
