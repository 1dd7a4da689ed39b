"""The force kernel's blocks (128 consecutive sites, both parities and all
directions) at their edges against the oracle: lattices of less than a block,
a partial last block, thin extents, an F that starts 8 bytes into a line, and
accumulation into F and G."""
import pytest

from oracle import oracle as O
from paper_1311_4462_amd import inputs

from .gpu_util import from_native, oparams, rel, to_native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 2, 10, 4), (4, 6, 4, 8)])
@pytest.mark.parametrize("flavor,recon,prec", [(2, 12, 1), (1, 18, 1), (-1, 12, 0)])
def test_force_blocks(dims, flavor, recon, prec):
    import torch

    from paper_1311_4462_amd import api
    ctx = api.Context()
    p = api.make_params(dims, 0.16, 0.14, 0.18 if flavor == 2 else 0.0, flavor)
    op = oparams(p)
    U = inputs.gauge_field(dims, "haar", 351)
    X = O.project(inputs.gaussian_spinor(dims, op.nf, 352), dims, 0)
    g = api.Gauge(ctx, U, p, recon=recon, precs=(prec,))
    x = to_native(api, ctx, X, p, prec, 0)
    Fref, Gref = O.force(op, U, from_native(api, ctx, x, p, prec, 0)[0], "asym")
    dt = torch.complex128 if prec == 0 else torch.complex64
    buf = torch.zeros(U.size + 1, dtype=dt, device="cuda")
    F = buf[1:].reshape(U.shape)
    G = torch.zeros(U.shape, dtype=dt, device="cuda")
    api.tm_force(ctx, F, prec, x, g, prec, 0, 1.0, False, G)
    api.tm_force(ctx, F, prec, x, g, prec, 0, 0.5, True, G)
    tol = 1e-10 if prec == 0 else 1e-5
    assert rel(F.cpu().numpy(), 1.5 * Fref) < tol
    assert rel(G.cpu().numpy(), 1.5 * Gref) < tol
    assert buf[0].item() == 0
    g.close()
    ctx.close()
