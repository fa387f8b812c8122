"""Plane kernels of transform lengths 96 and 128: one plane per workgroup of
1024 threads, used from 96 planes of the three components on (FP64 planes of
128 stay rows and columns).  Both sides of each line of that rule, products
against the oracle (1e-12 in FP64, 1e-5 with FP32 transforms) and a solve whose
fused inner products they form, by the residual of the separate product."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import operator as op

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402

TOL = {V.VIE_FP64: 1e-12, V.VIE_MIXED: 1e-5}
# nz = 31 and 32: 93 and 96 planes; 128 and 129: 384 and 387
SHAPES = [(48, 37, 31), (48, 37, 32), (37, 48, 33), (48, 48, 48), (64, 49, 31), (49, 64, 32), (37, 37, 129), (40, 48, 128)]


@pytest.mark.parametrize("prec", [V.VIE_FP64, V.VIE_MIXED])
@pytest.mark.parametrize("shape", SHAPES)
def test_product(vie_ctx, shape, prec):
    case = W.random_tiny(sum(s * 41 ** i for i, s in enumerate(shape)), shape, fill=0.7)
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(7)
    x = rng.standard_normal((3,) + case.shape) + 1j * rng.standard_normal((3,) + case.shape)
    P = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                  ctx=vie_ctx)
    try:
        xd = torch.from_numpy(x).cuda()
        yd = torch.full_like(xd, complex("nan"))
        V.vie_matvec(P.handle, prec, xd, yd)
        torch.cuda.synchronize()
        got = yd.cpu().numpy()
    finally:
        P.close()
    want = op.matvec_fft(g, x * g.mask)
    assert np.all(got[:, ~g.mask] == 0)
    err = np.abs(got - want).max() / np.abs(want).max()
    assert err <= TOL[prec], err


@pytest.mark.parametrize("shape", [(48, 40, 32), (64, 50, 32)])
def test_solve(vie_ctx, shape):
    """The recursive residual of BiCGSTAB stays within a factor of ten of the
    true one at this tolerance."""
    case = W.random_tiny(11, shape, fill=0.8, spacing=(0.02, 0.02, 0.02))
    eps = np.where(case.eps == 1, 1.0 + 0j, 1.6 - 0.1j)
    case = dataclasses.replace(case, eps=eps)
    for prec, tol in ((V.VIE_FP64, 1e-9), (V.VIE_MIXED, 1e-7)):
        P = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                      ctx=vie_ctx)
        try:
            e = torch.from_numpy(V.vie_plane_wave(P.grid, (0, 0, 1), (1, 0, 0))).cuda()
            out, pol, ax = torch.empty_like(e), torch.empty_like(e), torch.empty_like(e)
            st = V.vie_stats()
            opts = V.make_opts(tol_outer=tol, maxit_outer=200, precondition=False, precision=prec)
            assert V.vie_solve_device(P.handle, e, opts, out, pol, st) == V.VIE_OK
            V.vie_matvec(P.handle, V.VIE_FP64, pol, ax)
            torch.cuda.synchronize()
            mask = torch.from_numpy(np.asarray(eps != 1)).cuda()
            res = torch.linalg.vector_norm((e - ax)[:, mask]) / torch.linalg.vector_norm(e[:, mask])
            assert float(res) <= 10 * tol, (prec, float(res))
        finally:
            P.close()


@pytest.mark.parametrize("prec", [V.VIE_FP64, V.VIE_MIXED])
@pytest.mark.parametrize("shape", [(24, 19, 1), (19, 24, 5), (32, 25, 3), (25, 32, 11)])
def test_plane_by_512_threads(vie_ctx, shape, prec):
    """Variant 1 of lengths 48 and 64 gives the bits of the 256-thread plane."""
    case = W.random_tiny(sum(s * 43 ** i for i, s in enumerate(shape)), shape, fill=0.7)
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(9)
    x = rng.standard_normal((3,) + case.shape) + 1j * rng.standard_normal((3,) + case.shape)
    P = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                  ctx=vie_ctx)
    got = {}
    try:
        xd = torch.from_numpy(x).cuda()
        for variant in (1, 2):
            V.vie_problem_set_plane(P.handle, prec, variant)
            yd = torch.full_like(xd, complex("nan"))
            V.vie_matvec(P.handle, prec, xd, yd)
            torch.cuda.synchronize()
            got[variant] = yd.cpu().numpy()
    finally:
        P.close()
    assert np.array_equal(got[1], got[2])
    want = op.matvec_fft(g, x * g.mask)
    assert np.abs(got[1] - want).max() / np.abs(want).max() <= TOL[prec]
