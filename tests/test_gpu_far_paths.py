"""The far field's two ways of summing, on both sides of the line between them
(shapes are (nz, ny, nx)): the matrix product at the edges of its tiles (16
rows, 32 mirror pairs of x, 16, 48 and 192 directions, several row tiles per
workgroup, several x parts) with directions enough that it is the faster one,
the direct sum on small boxes and few directions, and more directions than the
scratch holds at once in either.  Against the oracle's sum at the far field's
tolerance (1e-11); the entry point that allocates nothing gives the same bits."""
import numpy as np
import pytest

import workloads as W
from oracle import operator as op, physics, rooftop as rt

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402

PRODUCT = [((40, 40, 7), 400), ((33, 31, 8), 300), ((9, 40, 63), 192), ((20, 40, 65), 193), ((20, 30, 129), 49),
           ((64, 130, 5), 200), ((96, 96, 130), 16), ((20, 40, 7), 3000)]
DIRECT = [((1, 1, 1), 1), ((40, 2, 1), 5), ((16, 16, 16), 181), ((33, 64, 65), 2), ((128, 128, 1), 33), ((3, 1, 1), 180000)]


@pytest.mark.parametrize("rooftop", [False, True])
@pytest.mark.parametrize("shape,n_dir", PRODUCT + DIRECT)
def test_far_field(vie_ctx, shape, n_dir, rooftop):
    if rooftop and (n_dir > 1000 or shape[0] * shape[1] * shape[2] > 200000):
        pytest.skip("the collocated run covers the split and the large box")
    case = W.random_tiny(400 + shape[2], shape, fill=0.8, spacing=(0.04, 0.05, 0.03))
    if rooftop:
        case = W.padded(case)
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(401)
    P = rng.standard_normal((3,) + case.shape) + 1j * rng.standard_normal((3,) + case.shape)
    P = P * (rt.face_mask(g) if rooftop else g.mask)
    d = rng.standard_normal((n_dir, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    want = (rt if rooftop else physics).far_field_vector(g, P, d)
    Pr = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                   ctx=vie_ctx, rooftop=rooftop)
    try:
        x = torch.from_numpy(P).cuda()
        got = V.vie_far_field(Pr.handle, x, d)
        assert np.linalg.norm(got - want) <= 1e-11 * np.linalg.norm(want)
        if n_dir * -(-case.nx * case.ny * case.nz // 2048) * 6 <= 1 << 20:
            f = torch.full((n_dir, 3), complex("nan"), dtype=torch.complex128, device="cuda")
            V.vie_far_field_noalloc(Pr.handle, x, n_dir, torch.from_numpy(d).cuda(), f)
            torch.cuda.synchronize()
            assert np.array_equal(f.cpu().numpy(), got)
    finally:
        Pr.close()


def test_kept_workspace_is_in_the_footprint(vie_ctx):
    """The device workspace that a problem keeps is counted and bounded by 16
    MiB; a context with a memory budget keeps none."""
    case = W.random_tiny(410, (24, 30, 20), fill=0.8)
    grid = V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength)
    rng = np.random.default_rng(411)
    d = rng.standard_normal((400, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    budgeted = V.vie_context_create(0, 4 << 30)
    try:
        for ctx in (vie_ctx, budgeted):
            P = V.Problem(grid, case.eps, None, 0, ctx=ctx)
            try:
                x = torch.ones(P.shape, dtype=torch.complex128, device="cuda")
                sizes = [P.info().footprint_bytes]
                for n in (1, 400, 7, 400):
                    V.vie_far_field(P.handle, x, d[:n])
                    sizes.append(P.info().footprint_bytes)
                kept = [s - sizes[0] for s in sizes[1:]]
                if ctx == budgeted:
                    assert kept == [0, 0, 0, 0]
                else:
                    assert 9 * 8 <= kept[0] < kept[1] == kept[2] == kept[3] <= 16 << 20 and kept[1] >= 400 * 9 * 8
            finally:
                P.close()
    finally:
        V.vie_context_destroy(budgeted)
