"""Cases of the library's device paths on the CPU emulation build, run in a
child process started with emu_env():

    python tests/emu/paths.py LIB CASE
"""
from __future__ import annotations

import ctypes as C
import os
import re
import sys
import tempfile

import numpy as np
import scipy.sparse as ssp

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


def _eval(c, w, est):
    """(value, gradient, last shape) of one evaluation, None for OOM."""
    try:
        v, g, _ = c.lml_grad(w.desc, w.x, w.y, w.h, est)
    except _lib.SdgpError as e:
        assert e.status == _lib.OOM, e
        return None
    return v, g, [c.get_option(k) for k in ("last_spmm_blocks", "last_update_blocks", "last_union_spmm")]


def _least_cap(lib, w, est, step=1.05):
    """The least workspace_cap (to the step) that one evaluation fits in."""
    cap = 1 << 15
    while True:
        c = EmuContext(lib)
        c.set_option("workspace_cap", cap)
        ok = _eval(c, w, est) is not None
        c.close()
        if ok:
            return cap
        cap = int(cap * step)


def case_cap(lib):
    """Under a workspace_cap a call that fits once fits again, with the same
    solver and bits, and whatever smaller calls came before it."""
    est = _lib.estimator(probes=4, seed=3, cg_rtol=1e-2, cg_max_iter=400, precond=1)
    w, s = small(n=130), small(n=70, seed=12)
    least = _least_cap(lib, w, est)
    print("least cap %d" % least)
    for f in (1.0, 1.4, 2.0, 3.0):
        cap = int(least * f)
        c = EmuContext(lib)
        c.set_option("workspace_cap", cap)
        a, b = _eval(c, w, est), _eval(c, w, est)
        print("cap %d: %s, again %s" % (cap, a and a[2], b and b[2]))
        assert a is not None and b is not None
        assert a[2] == b[2] and a[0] == b[0] and (a[1] == b[1]).all()
        c.close()
        c = EmuContext(lib)
        c.set_option("workspace_cap", cap)
        assert _eval(c, s, est) is not None and _eval(c, w, est) is not None, "after a smaller call"
        c.close()


def _store(lib, w, nnz, shape, lr=0):
    """Stores a tuned shape (spmm_blocks, update_blocks, union_spmm, fw_mfma)
    of the class of w's single evaluations with 1 to 32 probes."""
    n = w.x.shape[0]
    key = "emu-gfx950|u16|ni8|ns1|b1|n%d|r%d|lr%d|pc1" % (n.bit_length() - 1, round(2 * np.log2(nnz / n)), lr)
    c = EmuContext(lib)
    c.set_option("autotune", 2)
    assert c.lib.sdgp_tune_cache_put(None, key.encode(), (_lib.I64 * 4)(*shape)) == _lib.OK


def case_cap_lists(lib):
    """Under a workspace_cap the union lists that a call built are taken by the
    same call again, to the same bits."""
    est = _lib.estimator(probes=4, seed=3, cg_rtol=1e-2, cg_max_iter=400, precond=1)
    w = small(n=130)
    nnz = EmuContext(lib).kernel_nnz(w.desc, w.x, w.h)
    _store(lib, w, nnz, (8, 8, 1, 1))
    seen = set()
    for k in range(0, 12, 2):
        c = EmuContext(lib)
        c.set_option("autotune", 2)
        c.set_option("workspace_cap", int(400000 * 1.08 ** k))
        a, b = _eval(c, w, est), _eval(c, w, est)
        print("cap %d: %s, again %s" % (c.get_option("workspace_cap"), a and a[2], b and b[2]))
        assert c.get_option("last_tuned") == 1
        if a is not None:
            seen.add(a[2][2])
            assert b is not None and a[2] == b[2] and a[0] == b[0] and (a[1] == b[1]).all()
        c.close()
    assert seen == {0, 1}                   # caps on both sides


def _traced(call):
    """The launches of call() as (kernel, grid x, grid y, grid z)."""
    with tempfile.TemporaryFile() as f:
        sys.stderr.flush()
        old = os.dup(2)
        os.dup2(f.fileno(), 2)
        os.environ["EMU_TRACE"] = "1"
        try:
            call()
        finally:
            del os.environ["EMU_TRACE"]
            os.dup2(old, 2)
            os.close(old)
        f.seek(0)
        text = f.read().decode()
    return [(m[0], int(m[1]), int(m[2]), int(m[3]))
            for m in re.findall(r"\[hipemu\] (\S.*?) grid \((\d+),(\d+),(\d+)\)", text)]


def case_refused_trial(lib):
    """The tuner times no candidate whose union lists the workspace_cap refuses
    (one step of CSR rows has 16 rows, of the lists 64: at 130 points 16 blocks
    and 8)."""
    est = _lib.estimator(probes=4, seed=3, cg_rtol=1e-8, cg_max_iter=400, precond=1)
    w = small(n=130)
    forms = {}
    for cap in (0, 470000):
        c = EmuContext(lib)
        c.set_option("autotune", 2)
        c.set_option("workspace_cap", cap)
        os.environ["SDGP_TUNE_CACHE"] += "x"
        lines = _traced(lambda: c.lml_grad(w.desc, w.x, w.y, w.h, est))
        forms[cap] = {ln[:2] for ln in lines if ln[0].startswith("k_cg_spmm")}
        print("cap %d: %s" % (cap, sorted(forms[cap])))
    assert forms[0] == {("k_cg_spmm<1>", 16), ("k_cg_spmm_u<1, false>", 8)}
    assert forms[470000] == {("k_cg_spmm<1>", 16)}


def case_csr_grid(lib):
    """The SpMM over CSR rows has its own grid (16 rows a step) where the union
    lists' (64 rows a step) does not apply: when column 0 goes alone after the
    lists, and when tuned lists do not fit."""
    w = small(n=400)
    c = EmuContext(lib)
    c.set_option("union_spmm", 1)
    est = _lib.estimator(probes=1, seed=3, cg_rtol=1e-9, probe_rtol=1e-1, cg_max_iter=400, precond=1)
    lines = _traced(lambda: c.lml_grad(w.desc, w.x, w.y, w.h, est))
    grids = {ln[:2] for ln in lines if ln[0].startswith("k_cg_spmm")}
    print("alone for %d iterations: %s" % (c.get_option("last_y_tail"), sorted(grids)))
    assert c.get_option("last_y_tail") > 0
    assert grids == {("k_cg_spmm_u<1, false>", 8), ("k_cg_spmm<0>", 32)}
    v, g, _ = c.lml_grad(w.desc, w.x, w.y, w.h, est)
    c.set_option("union_spmm", 0)
    v0, g0, _ = c.lml_grad(w.desc, w.x, w.y, w.h, est)
    assert abs(v - v0) <= 1e-9 * abs(v0) and np.abs(g - g0).max() <= 1e-7 * np.abs(g0).max()

    w = small(n=130)
    _store(lib, w, EmuContext(lib).kernel_nnz(w.desc, w.x, w.h), (8, 8, 1, 1))
    est = _lib.estimator(probes=4, seed=3, cg_rtol=1e-2, cg_max_iter=400, precond=1)
    for cap, shape in ((0, [8, 8, 1]), (470000, [16, 8, 0])):
        c = EmuContext(lib)
        c.set_option("autotune", 2)
        c.set_option("workspace_cap", cap)
        got = _eval(c, w, est)[2]
        print("cap %d: %s" % (cap, got))
        assert got == shape and c.get_option("last_tuned") == 1


def sides(n=820, noise=4.0):
    """A population whose members lie on both sides of the column CG's rule (the
    first: every pair stored) and the same with an invalid first member."""
    w = small(n=n, n1=2)
    p = wl.unpack_hyper(w.desc, w.h)
    one = lambda s2, rc: wl.pack_hyper(w.desc, s2, rc, p["a"], p["beta"], p["r"], p["c"], noise)
    H = np.array([one(0.7, 2.0), one(1.0, p["r_core"]), one(0.5, 2.0), one(1.2, 0.8 * p["r_core"])])
    bad = H.copy()
    bad[0, 0] = bad[2, 0] = -1.0
    return w, H, bad


def case_sides(lib):
    """Members take the solver that their own entries call for: what the others
    store does not change their bits."""
    w, H, bad = sides()
    est = _lib.estimator(probes=2, seed=3, cg_rtol=1e-3, cg_max_iter=200, precond=1)
    c = EmuContext(lib)
    v, g, st, info = c.lml_grad_batched(w.desc, w.x, w.y, H, est)
    print("entries %s, blocks %d" % ([i.nnz for i in info], c.get_option("last_update_blocks")))
    assert (st == 0).all() and c.get_option("last_update_blocks") > 0
    v1, g1, st1, _ = c.lml_grad_batched(w.desc, w.x, w.y, bad, est)
    assert list(st1) == [_lib.INVALID_ARG, 0, _lib.INVALID_ARG, 0] and c.get_option("last_update_blocks") == 0
    assert (v[1::2] == v1[1::2]).all() and (g[1::2] == g1[1::2]).all()
    for m in (0, 2):                        # the largest core radius: the single call's order
        v1, g1, _ = c.lml_grad(w.desc, w.x, w.y, H[m], est)
        assert v[m] == v1 and (g[m] == g1).all()


def case_canonical(lib):
    """Caller-order CSR with rows past the rank sort's 512 entries.  Up to a
    quarter of them: the short rows are ranked and the segmented sort sees the
    long ones alone; more: all rows are sorted.  Either way the result is the
    sorted-order assembly in the caller's order."""
    k = 530                                 # a clique of points under one bump
    for n in (4 * k + 3, 4 * k, 4 * k - 1):
        rng = np.random.default_rng(5)
        x = 0.6 + 0.4 * rng.random((n, 2))
        x[rng.permutation(n)[:k]] = 0.25 + 0.01 * rng.random((k, 2))
        d = wl.KernelDesc(2, 1, 1, 0, 1)
        h = wl.pack_hyper(d, 1.0, 0.03, np.full((1, 1), 0.7), np.ones((1, 1)), np.full((1, 1), 0.05),
                          np.full((1, 1, 2), 0.255), 1e-2)
        c = EmuContext(lib)
        nnz = c.kernel_nnz(d, x, h)
        srp, scol, sval, perm = c.kernel_assemble_sorted(d, x, h, nnz)
        rp, col, val = np.zeros(n + 1, dtype=np.int64), np.zeros(nnz, dtype=np.int32), np.zeros(nnz)
        out, dd = _lib.I64(0), _lib.desc_of(d)
        lines = _traced(lambda: c._check(c.lib.sdgp_kernel_assemble(
            c.h, C.byref(dd), x.ctypes.data, n, h.ctypes.data, 1, rp.ctypes.data, col.ctypes.data, val.ctypes.data,
            nnz, C.byref(out))))
        rows = perm[np.repeat(np.arange(n), np.diff(srp))]
        order = np.lexsort((perm[scol], rows))
        assert out.value == nnz and (np.diff(rp) > 512).sum() == k
        assert (rp[1:] == np.cumsum(np.bincount(rows, minlength=n))).all() and rp[0] == 0
        assert (col == perm[scol][order]).all() and (val == sval[order]).all()
        grids = {ln[0]: ln[1] for ln in lines if ln[0].startswith("k_canon")}
        print("canonical %d rows, %d long: %s" % (n, k, grids))
        split = n >= 4 * k
        assert grids.get("k_canon_rank") == ((n + 3) // 4 if split else None)
        assert grids["k_canon_copy"] == ((k if split else n) + 3) // 4


def case_block_members(lib):
    """The block CG over several members that stop at different iterations, over
    CSR rows and over union lists (with few update blocks: with tile flags),
    against single solves and with its iterations replayed from a graph; and the
    replay of a solve whose y goes alone."""
    w = small(n=300)
    p = wl.unpack_hyper(w.desc, w.h)
    H = np.array([wl.pack_hyper(w.desc, s2, f * p["r_core"], p["a"], p["beta"], p["r"], p["c"], noise)
                  for s2, f, noise in ((1.0, 1.0, 1e-1), (0.3, 0.7, 3.0), (2.0, 0.8, 1.0))])
    for opts in ({"union_spmm": 0}, {"union_spmm": 1, "update_blocks": 4}):
        c = EmuContext(lib)
        for k, v in opts.items():
            c.set_option(k, v)
        est = _lib.estimator(probes=3, seed=3, cg_rtol=1e-6, cg_max_iter=900, precond=1)
        v, g, st, info = c.lml_grad_batched(w.desc, w.x, w.y, H, est)
        assert (st == 0).all() and c.get_option("last_update_blocks") > 0
        iters = [i.cg_iters for i in info]
        c.set_option("graph", 1)
        vg, gg, st, info = c.lml_grad_batched(w.desc, w.x, w.y, H, est)
        print("%s: iterations %s" % (opts, iters))
        assert len(set(iters)) == 3 and iters == [i.cg_iters for i in info]
        assert (v == vg).all() and (g == gg).all()
        c.set_option("graph", 0)
        for m in range(3):
            v1, g1, _ = c.lml_grad(w.desc, w.x, w.y, H[m], est)
            assert m > 0 or (v[m] == v1 and (g[m] == g1).all())
            assert abs(v[m] - v1) <= 1e-5 * abs(v1) and np.abs(g[m] - g1).max() <= 1e-4 * np.abs(g1).max()
        est = _lib.estimator(probes=3, seed=3, cg_rtol=1e-6, probe_rtol=3e-1, cg_max_iter=900, precond=1)
        v, g, _ = c.lml_grad(w.desc, w.x, w.y, H[0], est)
        alone = c.get_option("last_y_tail")
        c.set_option("graph", 1)
        vg, gg, _ = c.lml_grad(w.desc, w.x, w.y, H[0], est)
        print("  alone %d iterations" % alone)
        assert alone > 0 and alone == c.get_option("last_y_tail") and v == vg and (g == gg).all()


def case_few_rows(lib):
    """Products with an odd number of columns: a wavefront per row up to 12 rows a
    CU (256 CUs), four rows to a wavefront past it, far apart and shared up to 48
    where some rows are long; all give the product."""
    c = EmuContext(lib)
    for n, kernel in ((12 * 256, "k_spmm"), (12 * 256 + 1, "k_spmm_slab<kSpread>"),
                      (48 * 256, "k_spmm_slab<kSpread>"), (48 * 256 + 1, "k_spmm_slab<kRagged>")):
        for longest in (20, 700):
            rng = np.random.default_rng(n)
            lens = rng.integers(0, 20, n)
            lens[n // 3:n // 3 + n // 40] = longest
            rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
            col = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lens]).astype(np.int32)
            val, X = rng.standard_normal(len(col)), rng.standard_normal((n, 3))
            Y = np.zeros_like(X)
            lines = _traced(lambda: c._check(c.lib.sdgp_csr_spmm(c.h, n, rp.ctypes.data, col.ctypes.data,
                                                                 val.ctypes.data, X.ctypes.data, 3, Y.ctypes.data)))
            print(n, longest, lines)
            assert [ln[0] for ln in lines] == [kernel]
            S = ssp.csr_matrix((val, col, rp), shape=(n, n))
            assert (np.abs(Y - S @ X) <= 2e-13 * (abs(S) @ np.abs(X))).all()


def case_tile_flags(lib):
    """Tiles of F without bump values are flagged where F is wide: past 8 bump
    functions with the factored operator, past 16 with the assembled one."""
    est = lambda op: _lib.estimator(probes=1, seed=3, cg_rtol=1e-1, cg_max_iter=50, precond=1, operator_form=op)
    for n1, op, flags in ((8, 1, False), (9, 1, True), (16, 0, False), (17, 0, True)):
        w = small(n=70, n1=n1)
        c = EmuContext(lib)
        c.set_option("update_blocks", 1)
        names = {ln[0] for ln in _traced(lambda: c.lml_grad(w.desc, w.x, w.y, w.h, est(op)))}
        print(n1, op, "k_cg_ftiles" in names)
        assert ("k_cg_ftiles" in names) == flags


if __name__ == "__main__":
    globals()["case_" + sys.argv[2]](sys.argv[1])
    print("case %s holds" % sys.argv[2], flush=True)
