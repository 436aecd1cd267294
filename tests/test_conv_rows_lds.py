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


def test_planning_takes_no_time_per_image_row():
    """200 million rows: the plan is made in every call of a convolution."""
    import time
    from paper_2502_11407_amd import binding as gs
    p = gs.conv_problem("f16", 1, 1, 200000000, 1, 2, 3, 1, 1, 0)
    t0 = time.perf_counter()
    served = sum(gs.instance_schedule(i, p) is not None for i in range(gs.num_instances()))
    assert served > 0 and time.perf_counter() - t0 < 1.0
