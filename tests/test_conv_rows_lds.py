"""The LDS accesses of the row-staged convolution stay inside the workgroup's allocation: tests/conv_rows_lds.cpp walks
the windows of every lane, step and tile on the host, over the geometries of test_gpu_conv_rows.py and larger ones."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2502_11407_amd")


def test_every_lds_access_lies_inside_the_allocation(tmp_path):
    sys.path.insert(0, os.path.join(PKG, "csrc"))
    import build as kernel_build
    exe = str(tmp_path / "conv_rows_lds")
    r = subprocess.run([kernel_build.HIPCC] + kernel_build.FLAGS + ["-x", "hip", os.path.join(ROOT, "tests", "conv_rows_lds.cpp"), "-x", "none",
                        os.path.join(PKG, "libgensor.so"), "-Wl,-rpath," + PKG, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-1000:]
