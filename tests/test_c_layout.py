"""Every LDS read of the antidiagonal top merge, walked on the CPU with the kernel's own layout
functions: entries that fewer orders than the compiled bound do not have are read inside the
slab too."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_reads_stay_inside_their_slab(tmp_path):
    clang = "/opt/rocm/llvm/bin/clang++"
    cc = clang if os.path.exists(clang) else shutil.which("g++")
    exe = str(tmp_path / "driver")
    subprocess.check_call([cc, "-std=c++17", "-O1", "-I",
                           os.path.join(ROOT, "paper_2303_10672_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c_layout_driver.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 1_000_000
