"""Coarse-level kernels of the preconditioner at the edges of their tiles and
splits, against the oracle or plain linear algebra in FP64."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

import synth
from tests.helpers import box_problem, csr_close, random_heads, random_ks, weave_ks

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


# A one-level hierarchy applies the dense inverse of M itself: rows below, at
# and above the 64-row tiles, one to twelve tiles.  The inverse's error is
# kappa(M) eps; kappa <= 1e4 on these boxes (dt 10 s), FP32 rounds it to 6e-8
# per entry (sum of n terms).
@pytest.mark.parametrize("precision,tol", [(synth.FP64, 1e-10), (synth.MIXED, 1e-5)])
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 1, 1), (8, 8, 1), (13, 5, 1), (4, 4, 8), (43, 3, 1), (8, 8, 3),
                                   (11, 11, 6)])
def test_dense_inverse_tiles(rich, torch, shape, precision, tol):
    P = box_problem(*shape, dt=10.0)
    ks = random_ks(P, 41)
    s = rich.Solver(P, synth.Options(amg_max_levels=1, precision=precision), dev(torch, ks))
    for seed in (42, 43):  # set-up, then a refresh
        s.assemble(dev(torch, random_heads(P.n, seed, -70, -30)))
        assert s.levels() == 1
        rp, col, val = s.export_csr(rich.WHICH_A, 0)
        M = sp.csc_matrix(sp.csr_matrix((val, col, rp), shape=(P.n, P.n)))
        b = np.random.default_rng(seed).standard_normal(P.n)
        x = s.apply_prec(dev(torch, b)).cpu().numpy()
        xo = np.atleast_1d(spla.spsolve(M, b))
        assert np.linalg.norm(x - xo) <= tol * np.linalg.norm(xo)


# The refreshed coarse matrices are P^T A P of the refreshed fine ones (same
# terms; scipy adds them in another order: 1e-12 of the row maximum), on boxes
# with absent directions (the stencil's strides coincide) and with aggregates
# large enough that coarse rows pass the 32 entries summed in LDS at set-up.
@pytest.mark.parametrize("precision", [synth.FP64, synth.MIXED])
@pytest.mark.parametrize("shape,sweeps", [((40, 1, 1), 1), ((1, 1, 40), 3), ((1, 9, 7), 2), ((9, 1, 7), 3), ((2, 2, 9), 1),
                                          ((7, 9, 1), 3), ((21, 17, 13), 3), ((40, 37, 33), 6)])
def test_galerkin_refresh(rich, torch, shape, sweeps, precision):
    P = box_problem(*shape, dt=10.0)
    opts = synth.Options(amg_coarse_size=8, coarse_dense_max=8, amg_sweeps=sweeps, precision=precision)
    s = rich.Solver(P, opts, dev(torch, random_ks(P, 51)))
    longest = 0
    for seed in (52, 53, 54):
        s.assemble(dev(torch, random_heads(P.n, seed, -70, -30)))
        assert s.levels() >= 2
        rp, col, val = s.export_csr(rich.WHICH_A, 0)
        A = sp.csr_matrix((val, col, rp), shape=(P.n, P.n))
        for l in range(s.levels() - 1):
            agg, nc = s.export_aggregates(l)
            Pr = sp.csr_matrix((np.ones(A.shape[0]), (np.arange(A.shape[0]), agg)), shape=(A.shape[0], nc))
            C = sp.csr_matrix(Pr.T @ A @ Pr)
            rp, col, val = s.export_csr(rich.WHICH_A, l + 1)
            csr_close(rp, col, val, C, 1e-12)
            longest = max(longest, int(np.diff(rp).max()))
            A = sp.csr_matrix((val, col, rp), shape=(nc, nc))
    if sweeps == 6:
        assert longest > 32


# One V-cycle against the oracle's on the GPU's own M: coarse levels of every
# split of the aggregate-order kernels (short and long rows, aggregates of 2 to
# 64 rows, levels of one block up to several thousand, the l1-sweep coarsest
# level) and, where an aggregate outgrows their LDS, the separate kernels.
# FP64: the dense inverse's kappa eps; FP32: sums of a few hundred rounded terms.
@pytest.mark.parametrize("precision,tol", [(synth.FP64, 1e-10), (synth.MIXED, 1e-5)])
@pytest.mark.parametrize("shape,kw", [
    ((37, 5, 3), dict(amg_coarse_size=8, coarse_dense_max=8, amg_sweeps=1)),
    ((60, 1, 1), dict(amg_coarse_size=4, coarse_dense_max=8, amg_sweeps=2)),
    ((21, 17, 13), dict(amg_coarse_size=8, coarse_dense_max=64)),
    ((40, 37, 33), dict(amg_coarse_size=8, coarse_dense_max=8, amg_sweeps=6)),
    ((33, 31, 29), dict(amg_coarse_size=8, coarse_dense_max=8, amg_aggregation=1, amg_block=997)),
    ((150, 140, 130), dict()), ((150, 140, 130), dict(amg_max_levels=5))])
def test_vcycle_splits(rich, torch, orc, shape, kw, precision, tol):
    P = box_problem(*shape, dt=10.0)
    opts = synth.Options(precision=precision, **kw)
    s = rich.Solver(P, opts, dev(torch, random_ks(P, 61)))
    s.assemble(dev(torch, random_heads(P.n, 62, -70, -30)))
    rp, col, val = s.export_csr(rich.WHICH_A, 0)
    amg = orc.AMG(opts, sp.csr_matrix((val, col, rp), shape=(P.n, P.n)))
    assert s.levels() == amg.levels >= 3
    b = np.random.default_rng(63).standard_normal(P.n)
    x = s.apply_prec(dev(torch, b)).cpu().numpy()
    xo = amg.apply(b)
    assert np.linalg.norm(x - xo) <= tol * np.linalg.norm(xo)


# More rows than a launch of eight threads a row can hold (2^29 = 2^32 / 8): of a
# chain whose couplings (2 k + 1, 2 k + 2) are the strong ones, these match and the
# ends stay alone.
def test_match_sweep_many_rows(rich, torch):
    n = 2**29 + 4098
    e = torch.arange(3 * n, dtype=torch.int32, device="cuda")
    row, at = e // 3, e % 3 - 1
    del e
    strong = (at == 1) & (row % 2 == 1) | (at == -1) & (row % 2 == 0)
    val = torch.full((3 * n,), -0.1, dtype=torch.float64, device="cuda")
    val[strong] = -1.0
    val[at == 0] = 3.0
    row += at
    rowptr = torch.arange(n + 1, dtype=torch.int64, device="cuda").mul_(3).sub_(1)
    rowptr[0], rowptr[n] = 0, 3 * n - 2
    agg, nc = rich.match_sweep(rowptr, row[1:-1].clone(), val[1:-1].clone())
    assert nc == n // 2 + 1
    want = torch.arange(1, n + 1, dtype=torch.int32, device="cuda") // 2
    same = torch.equal(agg, want)
    del row, at, strong, val, rowptr, agg, want
    torch.cuda.empty_cache()
    assert same


def level_split(A, agg, nc, tsz):
    """(np, g, fits) of a smoothed level in aggregate order, from its matrix, aggregates
    and value size: blocks of np * 512 entries, g partial sums a row, and whether its
    largest block fits the LDS."""
    rows = np.diff(A.indptr)
    ent = np.bincount(agg, weights=rows, minlength=nc).astype(np.int64)
    most, nnz = int(ent.max()), A.nnz
    np_ = 4 if nnz >= (12 if tsz == 4 else 20) << 20 else 2 if nnz >= 5 << 17 else 1
    if np_ == 4 and most + 3 > 2048 - 256:
        np_ = 2
    align, run = (4, 256) if np_ == 4 else (2, 128)
    chunk = max(512 * np_ - most - align + 1, 256)
    first = np.concatenate([[0], np.cumsum(ent)])
    cut = np.append(np.searchsorted(first[:-1], np.arange(-(-nnz // chunk)) * chunk), nc)
    entries = int((first[cut[1:]] - first[cut[:-1]] // align * align).max())
    heads = np.concatenate([[0], np.cumsum(np.bincount(agg, minlength=nc))])
    mean = nnz // A.shape[0]
    g = 1 if mean < 8 else 2 if mean < 16 else 4 if mean < 32 else 8
    lds = (-(-entries // run) * run + int(np.diff(heads[cut]).max())) * tsz  # (np = 4: and the lists, at most 16 KB)
    return np_, g, lds <= 60 << 10


# The same on fibre fields, whose long rows and large aggregates reach what the boxes
# above do not: four and eight partial sums a row (chains of a lane group), blocks of
# 1024 entries, of 2048 with a column list, of 1024 where an aggregate is too long for
# the list's sort, and hierarchies that leave the aggregate order because a level does
# not fit, the first one or one behind others that do.  splits: of the levels smoothed,
# in FP64 and in FP32; None where one does not fit.
# One oracle hierarchy serves both precisions (it is built on the FP64 matrix).
@pytest.mark.parametrize("n,scale,kw,fp64,fp32", [
    (32, (1, 1e-2, 1e-4, 1e-2), dict(amg_sweeps=4), [(1, 8), (1, 2)], [(1, 8), (1, 2)]),
    (32, (1, 1e-2, 1e-4, 1e-4), dict(amg_sweeps=4), [(1, 4), (1, 4)], [(1, 4), (1, 4)]),
    (72, (1, 1e-2, 1e-4, 1e-2), dict(amg_sweeps=4, amg_max_levels=3), [(2, 8)], [(2, 8)]),
    (214, (1, 1e-2, 1e-4, 1e-2), dict(amg_sweeps=4, amg_max_levels=3), [(4, 8)], [(4, 8)]),
    (184, (1, 1e-2, 1e-4, 1e-2), dict(amg_sweeps=5, amg_max_levels=3), [(2, 8)], [(2, 8)]),
    (40, (1, 1e-2, 1e-6, 1e-9), dict(amg_sweeps=5), None, None),
    (32, (1, 1e-2, 1e-6, 1e-9), dict(amg_sweeps=6), None, [(1, 4), (1, 1)])])
def test_vcycle_long_rows(rich, torch, orc, n, scale, kw, fp64, fp32):
    P = box_problem(n, n, n, mean=synth.HARMONIC, dt=1e5)
    opts = dict(dict(amg_max_levels=4, amg_coarse_size=8, coarse_dense_max=8), **kw)
    ks, p = dev(torch, weave_ks(P, scale)), dev(torch, np.full(P.n, -50.0))
    b = np.random.default_rng(64).standard_normal(P.n)
    amg = None
    for precision, tol, want in ((synth.FP64, 1e-10, fp64), (synth.MIXED, 1e-5, fp32)):
        s = rich.Solver(P, synth.Options(precision=precision, **opts), ks)
        s.assemble(p)
        if amg is None:
            rp, col, val = s.export_csr(rich.WHICH_A, 0)
            amg = orc.AMG(synth.Options(**opts), sp.csr_matrix((val, col, rp), shape=(P.n, P.n)))
            L = [amg.level(l) for l in range(amg.levels)]
            xo = amg.apply(b)
        assert s.levels() == amg.levels
        got = [level_split(*L[l], L[l + 1][0].shape[0], 8 if precision == synth.FP64 else 4)
               for l in range(1, amg.levels - 1)]
        assert got and ([g[:2] for g in got] == want if want else not all(g[2] for g in got)), got
        x = s.apply_prec(dev(torch, b)).cpu().numpy()
        assert np.linalg.norm(x - xo) <= tol * np.linalg.norm(xo)
        s.assemble(p)  # and after a refresh
        assert np.array_equal(s.apply_prec(dev(torch, b)).cpu().numpy(), x)
        s.close()


# A set-up that fails (here on heads that are not numbers: no positive pivot in the
# coarsest matrix) leaves the handle without a hierarchy, and the next assembly builds
# one, as a new handle's does.
@pytest.mark.parametrize("precision", [synth.FP64, synth.MIXED])
@pytest.mark.parametrize("kw", [dict(), dict(amg_coarse_size=64), dict(amg_max_levels=1)])
def test_assembly_after_a_failed_setup(rich, torch, kw, precision):
    P = box_problem(12, 11, 9, dt=10.0)
    opts = synth.Options(precision=precision, **kw)
    ks, p = dev(torch, random_ks(P, 65)), random_heads(P.n, 66, -70, -30)
    b = dev(torch, np.random.default_rng(67).standard_normal(P.n))
    bad = p.copy()
    bad[P.n // 2] = np.nan
    s, fresh = rich.Solver(P, opts, ks), rich.Solver(P, opts, ks)
    with pytest.raises(rich.RichError) as e:
        s.assemble(dev(torch, bad))
    assert e.value.status == -9  # not positive definite
    assert s.levels() == 0
    with pytest.raises(rich.RichError) as e:
        s.apply_prec(b)
    assert e.value.status == -11  # not valid in this state
    for handle in (s, fresh):
        handle.assemble(dev(torch, p))
    assert s.levels() == fresh.levels()
    assert torch.equal(s.apply_prec(b), fresh.apply_prec(b))
    for handle in (s, fresh):
        handle.set_state(dev(torch, p))
    assert [t["gmres_its"] for t in s.step(1)] == [t["gmres_its"] for t in fresh.step(1)]
    assert torch.equal(s.get_state(), fresh.get_state())
