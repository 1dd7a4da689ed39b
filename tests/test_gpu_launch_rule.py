"""Launch shapes outside the tuned sizes: the rule's choice for every link
format and precision exists and gives the operator, and a tuner's file is read
only for launches like the one it was timed on."""
import pytest

from oracle import oracle as O
from paper_1311_4462_amd import inputs

from .gpu_util import TOL, check_solve, from_native, oparams, oracle_dslash, rel, to_native

pytestmark = pytest.mark.gpu

CSW = 1.57


@pytest.fixture
def api():
    from paper_1311_4462_amd import api as a
    return a


# 8, 192 and 960 sites per parity, untuned
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 6), (8, 6, 4, 10)])
@pytest.mark.parametrize("flavor", [1, -1, 2])
def test_small_clover_with_18_real_links(api, dims, flavor):
    c = api.Context()
    p = api.make_params(dims, 0.16, 0.13, 0.17 if flavor == 2 else 0.0, flavor, csw=CSW)
    U = inputs.gauge_field(dims, "haar", 401)
    op = O.with_clover(oparams(p), U, CSW)
    g = api.Gauge(c, U, p, recon=18, precs=(0, 1))
    a = O.project(inputs.gaussian_spinor(dims, op.nf, 402, nrhs=2), dims, 0)
    xv = O.project(inputs.gaussian_spinor(dims, op.nf, 403, nrhs=2), dims, 1)
    for prec in (0, 1):
        t, tx = to_native(api, c, a, p, prec, 0, 2), to_native(api, c, xv, p, prec, 1, 2)
        y = api.new_field(p, prec, 2)
        for pc in (0, 1):
            for dag in (0, 1):
                api.tm_mat_pc(c, y, t, g, prec, pc, dag, nrhs=2)
                got = from_native(api, c, y, p, prec, 0, 2)
                for r in range(2):
                    assert rel(got[r], O.mat_pc(op, U, a[r], ("asym", "sym")[pc], bool(dag))) < TOL[prec]
        for dag, twl, epi in ((0, 0, 1), (1, 1, 2), (1, 0, 4)):
            api.tm_dslash(c, y, t, g, prec, 1, dag, twl, epi, tx, -0.37, nrhs=2)
            got = from_native(api, c, y, p, prec, 1, 2)
            for r in range(2):
                assert rel(got[r], oracle_dslash(op, U, a[r], 1, dag, twl, epi, xv[r], -0.37)) < TOL[prec]
    tb = to_native(api, c, a, p, 0, 0, 2)
    for inner in (0, 1):
        x = api.new_field(p, 0, 2)
        res = api.tm_cg(c, x, tb, g, tol=1e-10, inner=inner, nrhs=2)
        xs = from_native(api, c, x, p, 0, 0, 2)
        for r in range(2):
            assert res[r]["status"] == 0
            check_solve(op, U, xs[r], a[r], "asym", res[r]["true_rel_res_normal"])
    g.close()
    c.close()


def test_tuner_tells_right_hand_sides_apart(api, monkeypatch, tmp_path):
    """One source and two on half the lattice are launches of their own to the tuner."""
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("TM_TUNE_CACHE", str(path))
    c = api.Context()
    c.set_tuning(True)
    keys = []
    for dims, nrhs in (((4, 4, 4, 16), 1), ((4, 4, 4, 8), 2), ((4, 4, 4, 4), 4)):
        p = api.make_params(dims, 0.16, 0.13, 0.0, 1)
        for prec in (0, 1, 2):
            g = api.Gauge(c, inputs.gauge_field(dims, "haar", 421), p, precs=(prec,))
            a = O.project(inputs.gaussian_spinor(dims, 1, 422, nrhs=nrhs), dims, 0)
            y = api.new_field(p, prec, nrhs)
            api.tm_mat_pc(c, y, to_native(api, c, a, p, prec, 0, nrhs), g, prec, 0, 0, nrhs=nrhs)
            g.close()
        keys.append({line.split()[0] for line in path.read_text().splitlines()})
    assert [len(k) for k in keys] == [6, 12, 18]
    c.close()


def _key(prec, nf, rhs, twl, recon, vh_total):
    return f"hop_p{prec}_f{nf}_{rhs}_d0_t{twl}_e0_c{recon}_v{vh_total}"


# shapes that no kernel has: two and four rhs per thread in FP32, 18-real links
# in blocks of 64, a group of rhs for one; bits as in the tuner's file
@pytest.mark.parametrize("prec,recon,nrhs,rhs,code", [
    (1, 12, 2, "r1", 256 | 1 << 18), (1, 12, 2, "r2", 256 | 1 << 18), (1, 12, 4, "r4", 256 | 2 << 18),
    (0, 18, 1, "r1", 64), (1, 12, 1, "r1", 512 | 1 << 13 | 4 << 20), (1, 18, 2, "n2", 512 | 1 << 13 | 2 << 20),
    (1, 12, 2, "n2", 256 | 1 << 18)])
def test_entry_of_another_launch_is_not_used(api, prec, recon, nrhs, rhs, code, monkeypatch, tmp_path):
    dims = (4, 4, 4, 4)
    p = api.make_params(dims, 0.16, 0.13, 0.0, 1)
    path = tmp_path / "tune.txt"
    path.write_text(f"{_key(prec, 1, rhs, 0, recon, 128 * nrhs)} {code}\n")
    monkeypatch.setenv("TM_TUNE_CACHE", str(path))
    c = api.Context()
    U = inputs.gauge_field(dims, "haar", 431)
    g = api.Gauge(c, U, p, recon=recon, precs=(prec,))
    a = O.project(inputs.gaussian_spinor(dims, 1, 432, nrhs=nrhs), dims, 1)
    y = api.new_field(p, prec, nrhs)
    api.tm_dslash(c, y, to_native(api, c, a, p, prec, 1, nrhs), g, prec, 0, nrhs=nrhs)
    got = from_native(api, c, y, p, prec, 0, nrhs)
    for r in range(nrhs):
        assert rel(got[r], oracle_dslash(oparams(p), U, a[r], 0, 0, 0, 0, None, 0.0)) < TOL[prec]
    g.close()
    c.close()


@pytest.mark.parametrize("split", ["0", "1"])
def test_forced_kernel_overrides_the_tuner_file(api, split, monkeypatch, tmp_path):
    """TM_HOP_SPLIT holds whatever the file says; the two kernels round the
    twist on load differently, so the bits of a hop tell which one ran."""
    dims = (6, 4, 4, 6)
    p = api.make_params(dims, 0.16, 0.13, 0.0, 1)
    U = inputs.gauge_field(dims, "haar", 441)
    a = O.project(inputs.gaussian_spinor(dims, 1, 442), dims, 1)
    path = tmp_path / "tune.txt"
    bits = []
    for forced, code in (("0", None), ("1", None), (split, (512 | 1 << 13, 256 | 1 << 16)[int(split)])):
        if code is not None:
            path.write_text(f"{_key(0, 1, 'r1', 1, 12, 288)} {code}\n")
            monkeypatch.setenv("TM_TUNE_CACHE", str(path))
        monkeypatch.setenv("TM_HOP_SPLIT", forced)
        c = api.Context()
        g = api.Gauge(c, U, p, precs=(0,))
        y = api.new_field(p, 0)
        api.tm_dslash(c, y, to_native(api, c, a, p, 0, 1), g, 0, 0, 0, 1)
        bits.append(from_native(api, c, y, p, 0, 0).tobytes())
        g.close()
        c.close()
    assert bits[0] != bits[1] and bits[2] == bits[int(split)]


@pytest.mark.parametrize("nr", ["-1", "-3", "0", "99"])
def test_group_outside_its_range(api, nr, monkeypatch):
    monkeypatch.setenv("TM_HOP_SPLIT", "1")
    monkeypatch.setenv("TM_HOP_NR", nr)
    dims, nrhs = (4, 4, 4, 6), 3
    c = api.Context()
    p = api.make_params(dims, 0.16, 0.13, 0.0, 1)
    U = inputs.gauge_field(dims, "haar", 451)
    g = api.Gauge(c, U, p, precs=(0,))
    a = O.project(inputs.gaussian_spinor(dims, 1, 452, nrhs=nrhs), dims, 1)
    y = api.new_field(p, 0, nrhs)
    api.tm_dslash(c, y, to_native(api, c, a, p, 0, 1, nrhs), g, 0, 0, nrhs=nrhs)
    got = from_native(api, c, y, p, 0, 0, nrhs)
    for r in range(nrhs):
        assert rel(got[r], oracle_dslash(oparams(p), U, a[r], 0, 0, 0, 0, None, 0.0)) < TOL[0]
    g.close()
    c.close()


# (lattice, flavours, precision, clover): sites on either side of the lines of the
# rule, 16-bit, FP32 and FP64
LINES = [((16, 16, 16, 32), 2, 2, 0), ((16, 16, 16, 36), 2, 2, 0), ((16, 16, 16, 36), 2, 3, 0),
         ((16, 16, 20, 36), 1, 2, 0), ((16, 20, 20, 32), 1, 3, 0),
         ((24, 24, 32, 56), 2, 1, 0), ((28, 28, 28, 48), 2, 1, 0),
         ((20, 20, 20, 60), 1, 0, 0), ((20, 20, 24, 56), 1, 0, 0),
         ((12, 16, 16, 28), 2, 0, 0), ((16, 16, 16, 24), 2, 0, 0), ((12, 16, 16, 40), 2, 0, 0),
         ((16, 16, 16, 32), 2, 0, 0), ((24, 24, 24, 72), 2, 0, 0), ((28, 28, 28, 48), 2, 0, 0),
         ((28, 28, 32, 64), 2, 0, 0), ((32, 32, 32, 60), 2, 0, 0),
         ((4, 4, 8, 8), 2, 1, 1), ((8, 8, 8, 8), 1, 1, 1), ((12, 12, 12, 20), 1, 0, 1), ((16, 16, 16, 12), 2, 0, 1)]


@pytest.mark.parametrize("recon", [12, 18, 8])
@pytest.mark.parametrize("dims,nf,prec,clover", LINES)
def test_rule_on_both_sides_of_its_lines(api, dims, nf, prec, clover, recon, monkeypatch):
    """The unforced launch and both forced kernels give the same operator (equal
    but for the rounding of the twist on load)."""
    import torch
    if clover and recon == 8:
        pytest.skip("no clover with 8-real links")
    p = api.make_params(dims, 0.16, 0.13, 0.17 if nf == 2 else 0.0, nf, csw=CSW * clover)
    small = torch.from_numpy(inputs.gauge_field((4, 4, 4, 4), "haar", 461)).cuda()
    U = small.repeat(1, *(n // 4 for n in dims[::-1]), 1, 1)
    gen = torch.Generator(device="cuda").manual_seed(462)
    a = torch.randn((1, *dims[::-1], nf, 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    outs = []
    for split in (None, "0", "1"):
        if split is not None:
            monkeypatch.setenv("TM_HOP_SPLIT", split)
        c = api.Context()
        g = api.Gauge(c, U, p, recon=recon, precs=(prec,))
        t = api.tm_spinor_pack(c, a, p, prec, 0, 1)
        for pc in (0, 1):
            for dag in (0, 1):
                y = api.new_field(p, prec)
                api.tm_mat_pc(c, y, t, g, prec, pc, dag)
                outs.append(api.tm_spinor_unpack(c, y, p, prec, 0, 1))
        g.close()
        c.close()
    for k in range(4):
        n = outs[k].norm().item()
        assert 0 < n < float("inf")
        for o in (outs[4 + k], outs[8 + k]):
            assert (o - outs[k]).norm().item() < (1e-14, 1e-6, 1e-3, 8e-3)[prec] * n
