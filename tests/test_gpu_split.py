"""Direction-split hop kernel (a wave per hop of 64 sites) against the oracle:
site counts around multiples of its 64-site blocks, extents that exercise the
coordinate division, every link format and precision, several right-hand sides
per block in even and ragged groups, and its reductions inside a solve."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1311_4462_amd import inputs

from .gpu_util import (TOL, check_solve, from_native, oparams, oracle_dslash, oracle_normal_residual, rel,
                       to_native)

pytestmark = pytest.mark.gpu


@pytest.fixture
def api():
    from paper_1311_4462_amd import api as a
    return a


# 8, 64, 288 and 840 sites per parity
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 2), (6, 4, 4, 6), (6, 10, 14, 2)])
@pytest.mark.parametrize("flavor,recon", [(1, 12), (-1, 18), (2, 12), (2, 8)])
def test_split_dslash(api, dims, flavor, recon, monkeypatch):
    monkeypatch.setenv("TM_HOP_SPLIT", "0")
    c0 = api.Context()                            # the one-thread kernel
    monkeypatch.setenv("TM_HOP_SPLIT", "1")
    monkeypatch.setenv("TM_HOP_ZC", "2" if dims[2] == 4 else "0")
    monkeypatch.setenv("TM_HOP_NR", "2")          # rhs per block: 2 + 1
    c = api.Context()
    p = api.make_params(dims, 0.16, 0.13, 0.17 if flavor == 2 else 0.0, flavor)
    op = oparams(p)
    U = inputs.gauge_field(dims, "haar", 301)
    g = api.Gauge(c, U, p, recon=recon, precs=(0, 1, 2, 3))
    nrhs = 3
    for out_par, prec in ((0, 0), (1, 1), (0, 2), (1, 3)):
        inp = O.project(inputs.gaussian_spinor(dims, op.nf, 302, nrhs=nrhs), dims, 1 - out_par)
        xv = O.project(inputs.gaussian_spinor(dims, op.nf, 303, nrhs=nrhs), dims, out_par)
        ti, tx = (to_native(api, c, a, p, prec, q, nrhs) for a, q in ((inp, 1 - out_par), (xv, out_par)))
        iq = from_native(api, c, ti, p, prec, 1 - out_par, nrhs)
        xq = from_native(api, c, tx, p, prec, out_par, nrhs)
        for dag, twl, epi in ((0, 0, 0), (1, 0, 1), (0, 0, 2), (1, 1, 3), (0, 1, 4), (1, 0, 5)):
            out = api.new_field(p, prec, nrhs)
            api.tm_dslash(c, out, ti, g, prec, out_par, dag, twl, epi, tx, -0.37, nrhs=nrhs)
            got = from_native(api, c, out, p, prec, out_par, nrhs)
            if recon == 8 and prec > 1:
                # rebuilding a link from 16-bit elements costs more than a hop's
                # tolerance against the oracle: the same links, one thread per site
                api.tm_dslash(c0, out, ti, g, prec, out_par, dag, twl, epi, tx, -0.37, nrhs=nrhs)
                assert rel(got, from_native(api, c0, out, p, prec, out_par, nrhs)) < TOL[prec]
                continue
            for r in range(nrhs):
                ref = oracle_dslash(op, U, iq[r], out_par, dag, twl, epi, xq[r], -0.37)
                assert rel(got[r], ref) < TOL[prec], (prec, dag, twl, epi, r)
    g.close()
    c.close()
    c0.close()


# right-hand sides and how many a block takes (FP32, FP64): one; all; 6 + 6 + 1
@pytest.mark.parametrize("nrhs,group", [(1, 1), (3, 3), (13, 6)])
@pytest.mark.parametrize("inner", [0, 1, 2])
def test_split_solve(api, nrhs, group, inner, monkeypatch):
    """A batched solve over two uneven lattices with the residual update and
    the norms in the direction-split kernel."""
    monkeypatch.setenv("TM_HOP_SPLIT", "1")
    monkeypatch.setenv("TM_HOP_NR", str(group))
    c = api.Context()
    probs = []
    for i, d in enumerate(((6, 4, 4, 8), (4, 6, 2, 6))):
        p = api.make_params(d, 0.15, 0.1, 0.0, 1)
        U = inputs.gauge_field(d, "haar", 310 + i)
        g = api.Gauge(c, U, p, precs=sorted({0, inner}))
        b = O.project(inputs.gaussian_spinor(d, 1, 320 + i, nrhs=nrhs), d, 0)
        probs.append((p, U, g, b, to_native(api, c, b, p, 0, 0, nrhs), api.new_field(p, 0, nrhs)))
    res = api.tm_cg_batched(c, [q[2] for q in probs], [q[5] for q in probs], [q[4] for q in probs],
                            [nrhs] * 2, tol=1e-10, inner=inner)
    for k, (p, U, g, b, _, x) in enumerate(probs):
        xs = from_native(api, c, x, p, 0, 0, nrhs)
        for r in range(nrhs):
            assert res[k * nrhs + r]["status"] == 0
            check_solve(oparams(p), U, xs[r], b[r], "asym", res[k * nrhs + r]["true_rel_res_normal"])
        g.close()
    c.close()


def test_rule_matches_forced(api, monkeypatch):
    """The launch rule's own choice and both forced kernels give the same
    operator (FP64, rounding apart) on a lattice of each side of its lines."""
    dims = (8, 6, 4, 10)
    outs = []
    for split in (None, "0", "1"):
        if split is not None:
            monkeypatch.setenv("TM_HOP_SPLIT", split)
        c = api.Context()
        for flavor, csw, recon in ((1, 0.0, 12), (2, 0.0, 18), (1, 1.2, 12)):
            p = api.make_params(dims, 0.16, 0.13, 0.17 if flavor == 2 else 0.0, flavor, csw=csw)
            g = api.Gauge(c, inputs.gauge_field(dims, "haar", 331), p, recon=recon, precs=(0,))
            a = O.project(inputs.gaussian_spinor(dims, 2 if flavor == 2 else 1, 332, nrhs=2), dims, 0)
            t = to_native(api, c, a, p, 0, 0, 2)
            for pc in (0, 1):
                for dag in (0, 1):
                    y = api.new_field(p, 0, 2)
                    api.tm_mat_pc(c, y, t, g, 0, pc, dag, nrhs=2)
                    outs.append(from_native(api, c, y, p, 0, 0, 2))
            g.close()
        c.close()
    n = len(outs) // 3
    for k in range(n):
        assert rel(outs[n + k], outs[k]) < 1e-14 and rel(outs[2 * n + k], outs[k]) < 1e-14
        assert np.isfinite(outs[k]).all()


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("flavor,recon,pc", [(1, 12, 0), (-1, 18, 1), (2, 12, 1), (2, 8, 0)])
def test_true_residual_in_the_hop(api, split, flavor, recon, pc, monkeypatch):
    """Reliable updates take c - M^+ M x from their last hop, rounded to the
    inner precision: the residual a mixed solve stops on (its last update's
    norm) is the oracle's, in every inner precision and both kernels."""
    monkeypatch.setenv("TM_HOP_SPLIT", str(split))
    c = api.Context()
    dims = (6, 4, 4, 6)
    p = api.make_params(dims, 0.15, 0.11, 0.13 if flavor == 2 else 0.0, flavor)
    op = oparams(p)
    U = inputs.gauge_field(dims, "near_unit", 341)
    g = api.Gauge(c, U, p, recon=recon, precs=(0, 1, 2, 3))
    b = O.project(inputs.gaussian_spinor(dims, op.nf, 342, nrhs=2), dims, 0)
    tb = to_native(api, c, b, p, 0, 0, 2)
    for inner in (1, 2, 3):
        x = api.new_field(p, 0, 2)
        res = api.tm_cg(c, x, tb, g, pc=pc, tol=1e-10, inner=inner, nrhs=2)
        xs = from_native(api, c, x, p, 0, 0, 2)
        for r in range(2):
            assert res[r]["status"] == 0 and res[r]["reliable_updates"] >= 2
            assert res[r]["precision_fallbacks"] == 0
            check_solve(op, U, xs[r], b[r], ("asym", "sym")[pc], res[r]["true_rel_res_normal"])
    g.close()
    c.close()


# vectors the last block of a launch finishes: by eight, four, two waves each,
# and by a wave each in two passes; 80 to 720 blocks in groups of up to 64
@pytest.mark.parametrize("nrhs", [1, 2, 3, 9])
def test_finish_in_the_hop(api, nrhs):
    """A mixed solve whose launches count their blocks in several groups: the
    residual it reports from its own reductions is that of its solution."""
    dims = (8, 8, 8, 20)
    c = api.Context()
    p = api.make_params(dims, 0.15, 0.1, 0.0, 1)
    U = inputs.gauge_field(dims, "haar", 341)
    g = api.Gauge(c, U, p, precs=(0, 1))
    b = O.project(inputs.gaussian_spinor(dims, 1, 342, nrhs=nrhs), dims, 0)
    x = api.new_field(p, 0, nrhs)
    res = api.tm_cg(c, x, to_native(api, c, b, p, 0, 0, nrhs), g, tol=1e-10, inner=1, nrhs=nrhs)
    xs = from_native(api, c, x, p, 0, 0, nrhs)
    for r in {0, nrhs - 1}:
        assert res[r]["status"] == 0 and res[r]["reliable_updates"] > 0
        check_solve(oparams(p), U, xs[r], b[r], "asym", res[r]["true_rel_res_normal"])
    g.close()
    c.close()


# a reliable update is due in iterations with and without the launches for it,
# in the last ones allowed, and for one right-hand side while another iterates
@pytest.mark.parametrize("inner", [1, 2, 3])
@pytest.mark.parametrize("graph,check", [(0, 0), (0, 3), (3, 0), (5, 0)])
def test_updates_between_iterations(api, inner, graph, check):
    """Whatever iteration a mixed solve ends on, the residual it reports is that
    of its solution; a free run converges."""
    dims, nrhs = (4, 4, 4, 6), 3
    c = api.Context()
    p = api.make_params(dims, 0.12, 0.1, 0.0, 1)
    U = inputs.gauge_field(dims, "haar", 351)
    g = api.Gauge(c, U, p, precs=(0, inner))
    b = O.project(inputs.gaussian_spinor(dims, 1, 352, nrhs=nrhs), dims, 0)
    b[1] = 0.0                       # converged from the start
    b[2].reshape(-1, 12)[1:] = 0.0   # a point source
    tb = to_native(api, c, b, p, 0, 0, nrhs)
    x = api.new_field(p, 0, nrhs)
    for m in (*range(1, 10), 500):
        res = api.tm_cg(c, x, tb, g, tol=1e-10, inner=inner, nrhs=nrhs, maxiter=m, graph_iters=graph,
                        check_every=check)
        xs = from_native(api, c, x, p, 0, 0, nrhs)
        assert not xs[1].any()
        assert m == 500 or res[0]["iters"] <= m
        for r in (0, 2):
            v = oracle_normal_residual(oparams(p), U, xs[r], b[r], "asym")
            assert abs(v - res[r]["true_rel_res_normal"]) <= 1e-3 * v, (m, r, v, res[r])
            if m == 500:
                assert res[r]["status"] == 0 and v <= 1.0000001e-10, (r, v)
    g.close()
    c.close()


def test_graph_of_small_blocks(api):
    """A captured FP64 doublet solve whose launches leave a partial per 32 sites,
    more than a BLAS launch: every buffer exists before the capture."""
    import torch
    dims = (16, 16, 32, 66)
    c = api.Context()
    p = api.make_params(dims, 0.1, 0.1, 0.05, 2)
    U = torch.zeros((4, *dims[::-1], 3, 3), dtype=torch.complex128, device="cuda")
    U[..., range(3), range(3)] = 1.0
    g = api.Gauge(c, U, p, precs=(0,))
    b = torch.randn((1, *dims[::-1], 2, 4, 3), dtype=torch.complex128, device="cuda")
    x = api.new_field(p, 0, 1)
    res = api.tm_cg(c, x, api.tm_spinor_pack(c, b, p, 0, 0, 1), g, tol=1e-6, graph_iters=2)
    assert res[0]["status"] == 0 and res[0]["true_rel_res_normal"] <= 1e-6
    g.close()
    c.close()
