"""Plane kernels of transform lengths 96 and 128 (a workgroup of 1024 threads
per plane) and of 48 and 64 by 512 threads, on boxes whose x and y transforms
are equal (shapes are (nz, ny, nx)): both sides of every line of the rule that
picks them, products against the oracle (1e-12 in FP64, 1e-5 with FP32
transforms), solves whose fused updates and inner products they form, and
batches against the same right-hand sides alone, bit for bit.

Which kernels ran shows in the pass times where the planes are long: the column
passes of a product on planes are empty.  Up to 64 every square box is on them."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import operator as op

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402

TOL = {V.VIE_FP64: 1e-12, V.VIE_MIXED: 1e-5}
# shape, length, on planes in (FP64, mixed)
LINES = [((31, 37, 48), 96, (False, False)), ((32, 48, 37), 96, (True, True)), ((48, 48, 48), 96, (True, True)),
         ((85, 37, 40), 96, (True, True)), ((86, 40, 37), 96, (False, False)), ((136, 37, 38), 96, (False, False)),
         ((137, 38, 37), 96, (True, False)), ((172, 37, 37), 96, (False, False)),
         ((31, 49, 64), 128, (False, False)), ((32, 64, 49), 128, (False, True)), ((85, 49, 49), 128, (False, True)),
         ((86, 49, 50), 128, (False, False)), ((106, 49, 49), 128, (False, False)), ((107, 50, 49), 128, (False, True))]


def _problem(ctx, case):
    return V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                     ctx=ctx)


def _product(P, prec, x):
    xd = torch.from_numpy(x).cuda()
    yd = torch.full_like(xd, complex("nan"))
    V.vie_matvec(P.handle, prec, xd, yd)
    torch.cuda.synchronize()
    return yd.cpu().numpy()


def _on_planes(P, prec):
    x = torch.zeros(P.shape, dtype=torch.complex128, device="cuda")
    ms = np.min([V.vie_matvec_profile(P.handle, prec, x, torch.empty_like(x), 10) for _ in range(3)], axis=0)
    ratio = (ms[1] + ms[3]) / (ms[0] + ms[4])   # 0.4 and less on planes, 1.1 and more on rows and columns
    return bool(ratio < 0.75)


@pytest.mark.parametrize("prec", [V.VIE_FP64, V.VIE_MIXED])
@pytest.mark.parametrize("shape,length,planes", LINES)
def test_product_on_both_sides(vie_ctx, shape, length, planes, prec):
    case = W.random_tiny(sum(s * 41 ** i for i, s in enumerate(shape)), shape, fill=0.7)
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(7)
    x = rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)
    P = _problem(vie_ctx, case)
    try:
        assert (P.info().lx, P.info().ly) == (length, length)
        assert _on_planes(P, prec) == planes[prec]
        got = _product(P, prec, x)
    finally:
        P.close()
    want = op.matvec_fft(g, x * g.mask)
    assert np.all(got[:, ~g.mask] == 0)
    assert np.abs(got - want).max() <= TOL[prec] * np.abs(want).max()


@pytest.mark.parametrize("prec,tol", [(V.VIE_FP64, 1e-9), (V.VIE_MIXED, 1e-7)])
@pytest.mark.parametrize("shape,length", [((32, 40, 48), 96), ((32, 50, 64), 128), ((5, 24, 19), 48), ((5, 32, 25), 64)])
def test_solves_and_batches(vie_ctx, shape, length, prec, tol):
    """The recursive residual of BiCGSTAB stays within a factor of ten of the
    true one at these tolerances; systems of a batch equal those alone."""
    case = W.random_tiny(11, shape, fill=0.8, spacing=(0.02, 0.02, 0.02))
    eps = np.where(case.eps == 1, 1.0 + 0j, 1.6 - 0.1j)
    case = dataclasses.replace(case, eps=eps)
    P = _problem(vie_ctx, case)
    try:
        assert (P.info().lx, P.info().ly) == (length, length)
        if length > 64:
            assert _on_planes(P, prec) == (length != 128 or prec == V.VIE_MIXED)
        waves = [((0, 0, 1), (1, 0, 0)), ((0.6, 0, 0.8), (0.8, 0, -0.6)), ((0, 1, 0), (0, 0, 1j))]
        e = torch.from_numpy(np.stack([V.vie_plane_wave(P.grid, k, p) for k, p in waves])).cuda()
        out, pol, bout, bpol = (torch.empty_like(e) for _ in range(4))
        opts = V.make_opts(tol_outer=tol, maxit_outer=300, precondition=False, precision=prec)
        mask = torch.from_numpy(np.asarray(eps != 1)).cuda()
        ax = torch.empty_like(e[0])
        for r in range(len(waves)):
            assert V.vie_solve_device(P.handle, e[r], opts, out[r], pol[r], V.vie_stats()) == V.VIE_OK
            V.vie_matvec(P.handle, V.VIE_FP64, pol[r], ax)
            torch.cuda.synchronize()
            res = torch.linalg.vector_norm((e[r] - ax)[:, mask]) / torch.linalg.vector_norm(e[r][:, mask])
            assert float(res) <= 10 * tol
        assert V.vie_solve_batch(P.handle, len(waves), e, opts, bout, bpol) == V.VIE_OK
        torch.cuda.synchronize()
        assert torch.equal(bpol, pol) and torch.equal(bout, out)
    finally:
        P.close()


@pytest.mark.parametrize("prec", [V.VIE_FP64, V.VIE_MIXED])
@pytest.mark.parametrize("shape,length", [((1, 19, 24), 48), ((5, 24, 19), 48), ((3, 25, 32), 64), ((11, 32, 25), 64)])
def test_plane_by_512_threads(vie_ctx, shape, length, prec):
    """Variant 1 of lengths 48 and 64 gives the bits of the 256-thread plane."""
    case = W.random_tiny(sum(s * 43 ** i for i, s in enumerate(shape)), shape, fill=0.7)
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(9)
    x = rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)
    P = _problem(vie_ctx, case)
    got = {}
    try:
        assert (P.info().lx, P.info().ly) == (length, length)
        for variant in (1, 2):
            V.vie_problem_set_plane(P.handle, prec, variant)
            assert P.info().plane_variant[prec] == variant
            got[variant] = _product(P, prec, x)
    finally:
        P.close()
    assert np.array_equal(got[1], got[2])
    want = op.matvec_fft(g, x * g.mask)
    assert np.abs(got[1] - want).max() <= TOL[prec] * np.abs(want).max()
