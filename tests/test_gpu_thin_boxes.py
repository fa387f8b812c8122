"""Solves on boxes with an axis of one or two voxels: a row of two has the odd
transform length 3, whose first stage reads the padding too, so the fused
vector updates ahead of it have to write it.  A product with NaN input before
every solve leaves NaN in the LDS that the solve's workgroups get.

Bars: these operators' condition numbers are below 100, so a relative residual
of 1e-12 (FP64; mixed with refinement: 1e-9) puts the solution within 1e-10
(1e-7) of the dense one, and inner solves to 1e-10 (1e-4) the preconditioner
within 1e-8 (1e-2) of the exact block solves."""
import numpy as np
import pytest

import workloads as W
from oracle import krylov, operator as op, physics

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402

PRECS = [(V.VIE_FP64, 1e-12, 1e-10), (V.VIE_MIXED, 1e-9, 1e-7)]
WAVES = [((0.0, 0.0, 1.0), (1.0, 0.0, 0.0)), ((0.6, 0.0, 0.8), (0.8, 0.0, -0.6)), ((0.0, 1.0, 0.0), (0.0, 0.0, 1j))]
THIN = [(4, 5, 2), (5, 2, 4), (2, 4, 5), (3, 2, 2), (2, 2, 2), (6, 3, 1), (9, 30, 2)]   # (nz, ny, nx)


def _problem(ctx, case, blocks=None):
    grid = V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength)
    return V.Problem(grid, case.eps, blocks, 0 if blocks is None else int(blocks.max()) + 1, ctx=ctx)


@pytest.fixture(scope="module")
def dirty(vie_ctx):
    """Fills every CU's LDS with NaN, in either precision."""
    P = _problem(vie_ctx, W.random_tiny(1, (48, 40, 100), fill=0.9))
    x = torch.full((3, 48, 40, 100), complex("nan"), dtype=torch.complex128, device="cuda")
    y = torch.empty_like(x)
    yield lambda prec: V.vie_matvec(P.handle, prec, x, y)
    P.close()


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec,tol,bar", PRECS)
@pytest.mark.parametrize("shape", THIN)
def test_plain_and_batched_solves(vie_ctx, dirty, shape, prec, tol, bar):
    case = W.random_tiny(600 + 7 * shape[0] + shape[2], shape, fill=0.8, spacing=(0.03, 0.04, 0.05))
    g = op.Grid.from_case(case)
    want = np.stack([krylov.solve_dense(g, physics.plane_wave(g, k, p)) for k, p in WAVES])
    P = _problem(vie_ctx, case)
    try:
        e = torch.from_numpy(np.stack([V.vie_plane_wave(P.grid, k, p) for k, p in WAVES])).cuda()
        out, pol = torch.empty_like(e), torch.empty_like(e)
        opts = V.make_opts(tol_outer=tol, maxit_outer=2000, max_refine=6, precondition=False, precision=prec)
        for r in range(len(WAVES)):
            dirty(prec)
            assert V.vie_solve_device(P.handle, e[r], opts, out[r], pol[r], V.vie_stats()) == V.VIE_OK
        torch.cuda.synchronize()
        assert _rel(pol.cpu().numpy(), want) <= bar
        pol.zero_()
        dirty(prec)
        assert V.vie_solve_batch(P.handle, len(WAVES), e, opts, out, pol) == V.VIE_OK
        torch.cuda.synchronize()
        assert _rel(pol.cpu().numpy(), want) <= bar
    finally:
        P.close()


@pytest.mark.parametrize("flags", [0, V.VIE_FLAG_NO_BLOCK_KERNEL])
@pytest.mark.parametrize("prec,inner,bar", [(V.VIE_FP64, 1e-10, 1e-8), (V.VIE_MIXED, 1e-4, 1e-2)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_blocks_two_voxels_wide(vie_ctx, dirty, axis, prec, inner, bar, flags):
    """Blocks of two layers along one axis: the preconditioner against the
    oracle's, and a preconditioned solve against the dense solution."""
    case = W.random_tiny(650, (6, 6, 6), fill=0.9, spacing=(0.03, 0.04, 0.05))
    g = op.Grid.from_case(case)
    bid = np.where(g.mask, np.indices(case.shape)[axis] // 2, -1).astype(np.int32)
    rng = np.random.default_rng(651)
    w = (rng.standard_normal((3,) + case.shape) + 1j * rng.standard_normal((3,) + case.shape)) * g.mask
    want = krylov.BlockPreconditioner(g, bid, 3, 1e-12, 500)(w)
    P = _problem(vie_ctx, case, bid)
    try:
        wd = torch.from_numpy(w).cuda()
        yd = torch.empty_like(wd)
        dirty(prec)
        V.vie_precond_apply(P.handle, prec, inner, 500, wd, yd, flags=flags)
        torch.cuda.synchronize()
        assert _rel(yd.cpu().numpy(), want) <= bar
        e = torch.from_numpy(V.vie_plane_wave(P.grid, *WAVES[1])).cuda()
        out, pol = torch.empty_like(e), torch.empty_like(e)
        tol, field = (1e-12, 1e-10) if prec == V.VIE_FP64 else (1e-9, 1e-7)
        opts = V.make_opts(tol_outer=tol, tol_inner=1e-2, maxit_outer=500, max_refine=6, precision=prec, flags=flags)
        dirty(prec)
        assert V.vie_solve_device(P.handle, e, opts, out, pol, V.vie_stats()) == V.VIE_OK
        torch.cuda.synchronize()
        assert _rel(pol.cpu().numpy(), krylov.solve_dense(g, physics.plane_wave(g, *WAVES[1]))) <= field
    finally:
        P.close()
