"""CPU tests of options and stored choices that must not change a run's kernels."""

import os

from paper_1908_01719_amd import build
from paper_1908_01719_amd.binding import Simulator


def test_lds_option_selects_no_kernel(tmp_path):
    # The SpMV that option lds = 1 selected ended in a GPU memory fault. The
    # option and tuning lines that an earlier autotuner wrote with it are
    # accepted and the library holds no such kernel (kernel names stand in it
    # as text).
    with open(build.LIB, "rb") as f:
        lib = f.read()
    assert b"k_spmv_dot" in lib
    assert b"k_spmv_lds" not in lib
    path = os.path.join(str(tmp_path), "tuning.txt")
    with open(path, "w") as f:
        f.write("dmri-tuning-v1\ngfx950_cu256/0123456789abcdef/60/0/0/0 32 512 0 1 0.25\n")
    with Simulator(-1) as sim:
        for v in (1, 0):
            sim.set_options(lds=v)
            assert sim.dmri_get_option("lds") == v
        sim.dmri_load_tuning(path)
