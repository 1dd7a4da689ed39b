"""The course of a mixed solve: its iteration limit, and where its reliable
updates come."""
import pytest

from oracle import oracle as O
from paper_1311_4462_amd import inputs

from .gpu_util import to_native

pytestmark = pytest.mark.gpu


@pytest.fixture
def api():
    from paper_1311_4462_amd import api as a
    return a


def _mixed(api, inner, dims=(6, 4, 6, 8)):
    c = api.Context()
    p = api.make_params(dims, 0.15, 0.1, 0.0, 1)
    U = inputs.gauge_field(dims, "haar", 411)
    g = api.Gauge(c, U, p, precs=(0, inner))
    b = O.project(inputs.gaussian_spinor(dims, 1, 412), dims, 0)
    return c, g, to_native(api, c, b, p, 0, 0), api.new_field(p, 0)


@pytest.mark.parametrize("inner,graph", [(1, 3), (1, 4), (1, 8), (2, 2), (2, 5)])
def test_maxiter_counts_iterations_that_ran(api, inner, graph):
    """Tolerances between the iterated and the true residual of an iteration:
    the update that verifies it fails and the solve goes on.  It converges
    within as many iterations as it takes without a limit, although some of
    those enqueued did not run."""
    c, g, b, x = _mixed(api, inner)
    kw = dict(inner=inner, graph_iters=graph)
    went_on = 0
    for m in range(5, 60):
        r = api.tm_cg(c, x, b, g, tol=1e-13, maxiter=m, **kw)[0]
        if r["status"] == 0:
            break
        it, true = r["res_history"][-1], r["true_rel_res_normal"]
        if not it * (1 + 1e-9) < true < 1.5 * it:
            continue
        tol = (it * true) ** 0.5
        free = api.tm_cg(c, x, b, g, tol=tol, **kw)[0]
        assert free["status"] == 0
        went_on += free["iters"] > m
        r = api.tm_cg(c, x, b, g, tol=tol, maxiter=free["iters"], **kw)[0]
        assert r["status"] == 0 and r["iters"] == free["iters"], (m, tol, r)
    assert went_on >= 3
    g.close()
    c.close()


@pytest.mark.parametrize("inner", [1, 2, 3])
@pytest.mark.parametrize("every", [2, 5, 8])
def test_unconverged_solve_ran_all_it_may(api, inner, every):
    c, g, b, x = _mixed(api, inner)
    for k in range(20):
        tol = 10.0 ** (-4 - k / 3)
        n = api.tm_cg(c, x, b, g, tol=tol, inner=inner, check_every=every)[0]["iters"]
        for m in range(max(1, n - 3), n + 1):
            r = api.tm_cg(c, x, b, g, tol=tol, inner=inner, check_every=every, maxiter=m)[0]
            assert r["status"] == 0 or r["iters"] == m, (tol, m, r)
    g.close()
    c.close()


@pytest.mark.parametrize("inner", [1, 2, 3])
def test_given_delta_places_the_updates(api, inner):
    """With a threshold of the caller's the reliable updates follow the
    iteration that reaches it: the same course under any host period."""
    import torch
    c, g, b, x = _mixed(api, inner)
    runs = []
    for kw in (dict(check_every=1), dict(check_every=3), dict(), dict(graph_iters=5)):
        r = api.tm_cg(c, x, b, g, tol=1e-10, inner=inner, delta=0.05, **kw)[0]
        assert r["status"] == 0
        runs.append((r["iters"], r["reliable_updates"], x.clone()))
    for it, up, v in runs[1:]:
        assert (it, up) == runs[0][:2] and torch.equal(v, runs[0][2])
    g.close()
    c.close()
