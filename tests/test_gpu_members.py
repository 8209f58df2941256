"""Populations whose members take different solvers, and populations and graph
replays of the block CG (a launch-shape option asks for it, where small point
sets would take the column CG)."""
import numpy as np
import pytest

from paper_2205_09070_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def test_members_on_both_sides_of_the_column_rule():
    """Two members store every pair (block CG), two a few neighbours (column
    CG).  The sparse ones' bits are those of the batch whose dense members are
    invalid, the dense ones' those of a single call (their core radius is the
    population's largest), and all agree with single calls to the bounds of the
    batched-against-single test."""
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w = wl.random_small(1000, 2, 3, 2, 31, combine=1, per_row=12.0, noise_var=1e-2)
    p = wl.unpack_hyper(w.desc, w.h)
    H = np.array([wl.pack_hyper(w.desc, s2, rc, p["a"], p["beta"], p["r"], p["c"], 0.5)
                  for s2, rc in ((0.7, 2.0), (1.0, p["r_core"]), (0.5, 2.0), (1.2, 0.8 * p["r_core"]))])
    bad = H.copy()
    bad[[0, 2], 0] = -1.0
    est = sd.estimator(probes=8, seed=3, cg_rtol=1e-11, cg_max_iter=3000, precond=1)
    gu.log("members on both sides")
    c = gu.ctx()
    x, y = gu.dev(w.x), gu.dev(w.y)
    v, g, st, info = c.lml_grad_batched(w.desc, x, y, H, est)
    gu.log("  entries %s" % [i.nnz for i in info])
    assert (st == sd.OK).all() and c.get_option("last_update_blocks") > 0
    v1, g1, st1, _ = c.lml_grad_batched(w.desc, x, y, bad, est)
    assert c.get_option("last_update_blocks") == 0
    assert list(st1) == [sd.INVALID_ARG, sd.OK, sd.INVALID_ARG, sd.OK]
    assert np.array_equal(v[1::2], v1[1::2]) and np.array_equal(g[1::2], g1[1::2])
    for m in range(4):
        v1, g1, _ = c.lml_grad(w.desc, x, y, H[m], est)
        assert (c.get_option("last_update_blocks") > 0) == (m % 2 == 0)
        if m % 2 == 0:
            assert v[m] == v1 and np.array_equal(g[m], g1)
        assert abs(v[m] - v1) <= 1e-9 * abs(v1)
        assert gu.grad_close(g[m], g1, rel=1e-7).all()


def population(n, dim, n1, members, seed):
    """Members differ in variance, core radius and bump heights; the first has
    the largest core radius, so its single call shares the population's order."""
    w = wl.random_small(n, dim, n1, 2, seed, combine=1, per_row=14.0, noise_var=1e-2)
    rng = np.random.default_rng(seed)
    p = wl.unpack_hyper(w.desc, w.h)
    H = []
    for m in range(members):
        s2, f, a = (1.0, 1.0, 1.0) if m == 0 else (rng.uniform(0.2, 3.0), rng.uniform(0.5, 0.9), rng.uniform(0.3, 1.0))
        H.append(wl.pack_hyper(w.desc, s2, f * p["r_core"], a * p["a"], p["beta"], p["r"], p["c"],
                               p["noise_var"] * 10.0 ** rng.integers(0, 3)))
    return w, np.array(H)


@pytest.mark.parametrize("options", [{"union_spmm": 0}, {"union_spmm": 1}, {"union_spmm": 1, "update_blocks": 8},
                                     {"union_spmm": 0, "fw_mfma": 0}],
                         ids=["csr", "lists", "lists-tile-flags", "csr-broadcast"])
@pytest.mark.parametrize("n,dim,n1,probes,precond", [(3001, 3, 6, 12, 1), (1999, 2, 3, 40, 1), (2500, 2, 4, 8, 0)])
def test_block_members_match_single(options, n, dim, n1, probes, precond):
    """The block CG over several members that stop at different iterations (the
    launch grid shrinks as they do), their lists and tile flags side by side:
    every member against its single block CG solve."""
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w, H = population(n, dim, n1, 5, 40 + n1)
    gu.log("block members n=%d %s" % (n, options))
    est = sd.estimator(probes=probes, seed=77, cg_rtol=1e-11, cg_max_iter=5000, precond=precond)
    c = gu.ctx()
    for k, v in options.items():
        c.set_option(k, v)
    x, y = gu.dev(w.x), gu.dev(w.y)
    v, g, st, infos = c.lml_grad_batched(w.desc, x, y, H, est)
    assert (st == sd.OK).all() and c.get_option("last_update_blocks") > 0
    assert c.get_option("last_union_spmm") == options["union_spmm"]
    iters = [i.cg_iters for i in infos]
    gu.log("  iterations %s" % iters)
    assert len(set(iters)) > 2
    for m in range(len(H)):
        v1, g1, i1 = c.lml_grad(w.desc, x, y, H[m], est)
        assert infos[m].nnz == i1.nnz
        if m == 0:
            assert v[m] == v1 and np.array_equal(g[m], g1)
        assert abs(v[m] - v1) <= 1e-9 * abs(v1)
        assert gu.grad_close(g[m], g1, rel=1e-7).all()


@pytest.mark.parametrize("union", [0, 1], ids=["csr", "lists"])
def test_block_invalid_member_fails_alone(union):
    gu.need_gpu()
    import paper_2205_09070_amd as sd
    w, H = population(2500, 2, 2, 4, 11)
    gu.log("block invalid member union=%d" % union)
    est = sd.estimator(probes=8, seed=9, cg_rtol=1e-11, cg_max_iter=5000)
    bad = H.copy()
    bad[2, 0] = -1.0
    c = gu.ctx()
    c.set_option("union_spmm", union)
    x, y = gu.dev(w.x), gu.dev(w.y)
    v, g, st, _ = c.lml_grad_batched(w.desc, x, y, bad, est)
    assert st[2] == sd.INVALID_ARG and np.isnan(v[2]) and np.isnan(g[2]).all()
    keep = [0, 1, 3]
    v1, g1, st1, _ = c.lml_grad_batched(w.desc, x, y, H[keep], est)
    assert c.get_option("last_update_blocks") > 0
    assert (st[keep] == sd.OK).all() and (st1 == sd.OK).all()
    assert np.array_equal(v[keep], v1) and np.array_equal(g[keep], g1)


@pytest.mark.parametrize("union", [0, 1], ids=["csr", "lists"])
@pytest.mark.parametrize("form", ["population", "factored", "alone"])
def test_block_graph_replay_is_bitwise(form, union):
    """Captured iterations (8 a graph) give bitwise the eager result of the block
    CG, on repeated calls with other stream work in between: a population whose
    active members shrink, the factored operator, and a solve whose y goes alone
    after its probes."""
    gu.need_gpu()
    import torch
    import paper_2205_09070_amd as sd
    w, H = population(3000, 3, 6, 4, 3)
    gu.log("block graph replay %s union=%d" % (form, union))
    est = sd.estimator(probes=12, seed=5, cg_rtol=1e-11, cg_max_iter=5000, precond=1,
                       operator_form=1 if form == "factored" else 0, probe_rtol=1e-3 if form == "alone" else 0.0)
    c = gu.ctx()
    c.set_option("union_spmm", union)
    x, y = gu.dev(w.x), gu.dev(w.y)

    def call():
        if form == "population":
            v, g, st, infos = c.lml_grad_batched(w.desc, x, y, H, est)
            assert (st == sd.OK).all()
            iters = [i.cg_iters for i in infos]
        else:
            v, g, info = c.lml_grad(w.desc, x, y, H[0], est)
            iters = [info.cg_iters]
        torch.cuda.synchronize()
        assert c.get_option("last_update_blocks") > 0
        assert (c.get_option("last_y_tail") > 0) == (form == "alone")
        return np.array(v), g, iters

    v0, g0, it0 = call()
    gu.log("  iterations %s" % it0)
    junk = torch.randn(1 << 20, dtype=torch.float64, device="cuda:0")
    c.set_option("graph", 1)
    for rep in range(3):
        junk.mul_(1.0001).add_(1.0)
        v1, g1, it1 = call()
        assert np.array_equal(v1, v0) and np.array_equal(g1, g0) and it1 == it0
