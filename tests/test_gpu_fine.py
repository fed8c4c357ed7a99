"""Fine-level kernels at the edges of their tiles and dispatch rules, against the
oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from tests.helpers import all_dirichlet, box_problem, csr_close, random_heads, random_ks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.fixture(scope="module")
def rich():
    import paper_2112_05051_amd as r
    r.load()
    return r


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# The marching kernels: 16 x 16 tiles with whole, single and missing columns, runs
# of one plane up to more than one block's 64, every side open, and heads that are
# not numbers or infinite reaching their neighbours and no further.  The laws and
# the sum of a row round about 20 times: 1e-12 of the largest entry.
@pytest.mark.parametrize("mean", [synth.ARITH, synth.UPSTREAM, synth.HARMONIC, synth.GEOMETRIC])
@pytest.mark.parametrize("shape", [(16, 16, 5), (17, 15, 4), (33, 32, 1), (2, 48, 70), (16, 1, 131)])
def test_marching_residual_and_assembly(rich, torch, orc, shape, mean):
    P = box_problem(*shape, mean=mean, dt=7.0)
    P.bc_type, P.bc_value = all_dirichlet()
    ks = random_ks(P, 71)
    p = random_heads(P.n, 72, saturated_fraction=0.05)
    th = orc.theta(P, random_heads(P.n, 73))
    s = rich.Solver(P, synth.Options(), dev(torch, ks))
    F_o = orc.residual(P, ks, p, th)
    F_g = s.residual(dev(torch, p), dev(torch, th)).cpu().numpy()
    assert np.max(np.abs(F_g - F_o)) <= 1e-12 * np.max(np.abs(F_o))
    s.assemble(dev(torch, p))
    csr_close(*s.export_csr(rich.WHICH_J), orc.jacobian(P, ks, p), 1e-12)
    csr_close(*s.export_csr(rich.WHICH_A, 0), orc.auxiliary(P, ks, p), 1e-12)
    p[P.n // 3], p[P.n // 2], p[-1] = np.nan, -np.inf, np.inf
    with np.errstate(all="ignore"):
        F_o = orc.residual(P, ks, p, th)
    F_g = s.residual(dev(torch, p), dev(torch, th)).cpu().numpy()
    ok = np.isfinite(F_o)
    assert np.array_equal(ok, np.isfinite(F_g)) and np.array_equal(np.isnan(F_o), np.isnan(F_g))
    assert np.max(np.abs(F_g[ok] - F_o[ok])) <= 1e-12 * np.max(np.abs(F_o[ok]))


# Theta with one and with four cells a thread (from 2^21 cells), remainders of both.
@pytest.mark.parametrize("shape", [(257, 1, 1), (1031, 45, 46)])
def test_theta_cells_per_thread(rich, torch, orc, shape):
    P = box_problem(*shape)
    p = random_heads(P.n, 81, saturated_fraction=0.05)
    s = rich.Solver(P, synth.Options(), dev(torch, np.full(P.n, synth.KS0)))
    th = s.theta(dev(torch, p)).cpu().numpy()
    th_o = orc.theta(P, p)
    assert np.max(np.abs(th - th_o)) <= 1e-13 * np.max(np.abs(th_o))


# On both sides of the 2^23 cells from which a thread takes four.
@pytest.mark.parametrize("shape", [(255, 257, 128), (257, 255, 129)])
def test_theta_on_both_sides(rich, torch, orc, shape):
    P = box_problem(*shape)
    p = random_heads(P.n, 82, saturated_fraction=0.05)
    s = rich.Solver(P, synth.Options(gmres_restart=1), torch.full((P.n,), synth.KS0, dtype=torch.float64, device="cuda"))
    th = s.theta(dev(torch, p)).cpu().numpy()
    th_o = orc.theta(P, p)
    assert np.max(np.abs(th - th_o)) <= 1e-13 * np.max(np.abs(th_o))


# Rows too short for the tiled smoother, on both sides of the 2^18 cells up to which
# one launch prolongates and smooths, and rows long enough for it; the result is
# stored straight into x, or through scratch where x is b or overlaps it.
@pytest.mark.parametrize("precision,tol", [(synth.FP64, 1e-10), (synth.MIXED, 1e-5)])
@pytest.mark.parametrize("shape", [(5, 4, 30), (47, 64, 87), (47, 64, 88), (64, 9, 6)])
def test_vcycle_result(rich, torch, orc, shape, precision, tol):
    P = box_problem(*shape, dt=10.0)
    opts = synth.Options(precision=precision, amg_coarse_size=64)
    s = rich.Solver(P, opts, dev(torch, random_ks(P, 91)))
    s.assemble(dev(torch, random_heads(P.n, 92, -70, -30)))
    rp, col, val = s.export_csr(rich.WHICH_A, 0)
    b = np.random.default_rng(93).standard_normal(P.n)
    xo = orc.AMG(opts, sp.csr_matrix((val, col, rp), shape=(P.n, P.n))).apply(b)
    x = s.apply_prec(dev(torch, b)).cpu().numpy()
    assert np.linalg.norm(x - xo) <= tol * np.linalg.norm(xo)
    for shift in (0, 8, -8):
        buf = torch.zeros(P.n + 8, dtype=torch.float64, device="cuda")
        bd, xd = (buf[max(0, -shift):], buf[max(0, shift):])
        bd[:P.n] = dev(torch, b)
        assert s._L.rich_apply_prec(s._h, bd.data_ptr(), xd.data_ptr()) == rich.OK
        assert np.array_equal(xd[:P.n].cpu().numpy(), x)


def same_values(g, o, rtol):
    """Not-numbers and infinities in the same places, finite values within rtol of the largest."""
    assert np.array_equal(np.isnan(g), np.isnan(o))
    inf = np.isinf(o)
    assert np.array_equal(np.isinf(g), inf) and np.array_equal(g[inf], o[inf])
    ok = np.isfinite(o)
    if ok.any():
        assert np.max(np.abs(g[ok] - o[ok])) <= rtol * max(np.max(np.abs(o[ok])), 1e-300)


def check_constants(rich, torch, orc, P, p, p_old):
    """Residual, J and M of the marching kernels where the grid's constants leave the usual range."""
    ks = random_ks(P, 74)
    th = orc.theta(P, p_old)
    s = rich.Solver(P, synth.Options(amg_max_levels=1, coarse_dense_max=0), dev(torch, ks))
    same_values(s.residual(dev(torch, p), dev(torch, th)).cpu().numpy(), orc.residual(P, ks, p, th), 1e-12)
    s.assemble(dev(torch, p))
    for which, ref in ((rich.WHICH_J, orc.jacobian), (rich.WHICH_A, orc.auxiliary)):
        rp, col, val = s.export_csr(which)
        R = sp.csr_matrix(ref(P, ks, p))
        R.sort_indices()
        assert np.array_equal(rp, R.indptr) and np.array_equal(col, R.indices)
        same_values(val, R.data, 1e-12)


# An infinite time step is the steady operator, and spacings whose square overflows
# switch a direction off: what is divided by them is zero.
@pytest.mark.parametrize("mean", [synth.ARITH, synth.UPSTREAM, synth.HARMONIC, synth.GEOMETRIC, synth.INTEGRAL])
@pytest.mark.parametrize("name", ["dt", "hx", "hy"])
def test_infinite_constants(rich, torch, orc, mean, name):
    P = box_problem(18, 17, 5, mean=mean, dt=7.0)
    setattr(P, name, np.inf if name == "dt" else 1e200)
    check_constants(rich, torch, orc, P, random_heads(P.n, 72, saturated_fraction=0.05), random_heads(P.n, 73))


# Constants so small that their reciprocal overflows: a saturated state that the
# time step leaves as it is, and heads that do not vary along y, divide to zero.
@pytest.mark.parametrize("mean", [synth.ARITH, synth.UPSTREAM, synth.HARMONIC, synth.GEOMETRIC, synth.INTEGRAL])
@pytest.mark.parametrize("name,value", [("dt", 1e-309), ("hy", 3e-155)])
def test_tiny_constants(rich, torch, orc, mean, name, value):
    P = box_problem(18, 17, 5, mean=mean, dt=7.0)
    setattr(P, name, value)
    p = np.repeat(np.random.default_rng(78).uniform(0.5, 5.0, (5, 1, 18)), 17, axis=1).reshape(-1)
    check_constants(rich, torch, orc, P, p, p)


# Flat grids: 32 x 8 tiles up to eight rows (whole, single and missing columns, more
# than one run of planes), and one thread per cell from 8192 cells on where x or y
# has one, from 32768 where it has two.
@pytest.mark.parametrize("mean", [synth.ARITH, synth.UPSTREAM, synth.HARMONIC, synth.GEOMETRIC])
@pytest.mark.parametrize("shape", [(32, 8, 5), (33, 7, 70), (17, 3, 1), (8191, 1, 1), (8192, 1, 1), (129, 2, 127), (2, 128, 128),
                                   (17, 9, 4)])
def test_flat_residual_and_assembly(rich, torch, orc, shape, mean):
    P = box_problem(*shape, mean=mean, dt=7.0)
    P.bc_type, P.bc_value = all_dirichlet()
    ks = random_ks(P, 75)
    p = random_heads(P.n, 76, saturated_fraction=0.05)
    th = orc.theta(P, random_heads(P.n, 77))
    s = rich.Solver(P, synth.Options(amg_max_levels=1, coarse_dense_max=0), dev(torch, ks))
    F_o = orc.residual(P, ks, p, th)
    F_g = s.residual(dev(torch, p), dev(torch, th)).cpu().numpy()
    assert np.max(np.abs(F_g - F_o)) <= 1e-12 * np.max(np.abs(F_o))
    s.assemble(dev(torch, p))
    csr_close(*s.export_csr(rich.WHICH_J), orc.jacobian(P, ks, p), 1e-12)
    csr_close(*s.export_csr(rich.WHICH_A, 0), orc.auxiliary(P, ks, p), 1e-12)
