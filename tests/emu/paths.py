"""Cases of the library's device paths on the CPU emulation build, run in a
child process started with emu_env():

    python tests/emu/paths.py LIB CASE
"""
from __future__ import annotations

import sys

from paper_2205_09070_amd import _lib
from paper_2205_09070_amd import workloads as wl
from tests.emu.emu_ctx import EmuContext


def small(n=200, n1=3, seed=11, per_row=12.0):
    return wl.random_small(n, 2, n1, 2, seed, combine=1, per_row=per_row, noise_var=1e-2)


def case_timing(lib):
    """With timing on, a solve without CG SpMM launches (column CG) reports
    none of them, also after a block CG solve on the same context."""
    w = small()
    c = EmuContext(lib)
    c.set_option("timing", 1)
    est = _lib.estimator(probes=4, seed=3, cg_rtol=1e-10, cg_max_iter=2000, precond=1)
    c.set_option("union_spmm", 0)
    _, _, block = c.lml_grad(w.desc, w.x, w.y, w.h, est)
    assert c.get_option("last_update_blocks") > 0
    assert block.spmm_launches >= block.cg_iters > 0 and block.spmm_ms > 0.0
    c.set_option("union_spmm", -1)
    _, _, col = c.lml_grad(w.desc, w.x, w.y, w.h, est)
    assert c.get_option("last_update_blocks") == 0
    print("block %d launches, column %d launches %.3f ms" % (block.spmm_launches, col.spmm_launches, col.spmm_ms))
    assert col.spmm_launches == 0 and col.spmm_ms == 0.0


if __name__ == "__main__":
    globals()["case_" + sys.argv[2]](sys.argv[1])
    print("case %s holds" % sys.argv[2], flush=True)
