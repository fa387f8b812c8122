"""The product's transforms read the lower half of a padded pencil only and
leave gaps in the LDS slots of rows: both edges of the boxes that share a
transform length, along each axis, against the oracle, with a product of large
values before it whose leftovers in the work buffer must not show.

Tolerance as for every product: 1e-12 in FP64, 1e-5 with FP32 transforms."""
import numpy as np
import pytest

import workloads as W
from oracle import operator as op

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402

TOL = {V.VIE_FP64: 1e-12, V.VIE_MIXED: 1e-5}
# fewest and most voxels of the transform lengths 8, 16, 32, 48, 64, 96, 128,
# 192 and 256: first radices 8, 16 and 4, last radices 16, 8, 4 and 3
EDGES = [(4, 4), (7, 8), (13, 16), (19, 24), (25, 32), (37, 48), (49, 64), (73, 96), (97, 128)]


@pytest.mark.parametrize("prec", [V.VIE_FP64, V.VIE_MIXED])
@pytest.mark.parametrize("edge", EDGES)
def test_half_empty_pencils(vie_ctx, edge, prec):
    few, most = edge
    shapes = {(most, few, 3), (few, most, 4), (5, 3, most), (most, 7, 2), (6, 9, few), (most, most, 2)}
    for shape in sorted(shapes):
        case = W.random_tiny(sum(s * 37 ** i for i, s in enumerate(shape)), shape, fill=0.7)
        g = op.Grid.from_case(case)
        rng = np.random.default_rng(most)
        x = rng.standard_normal((3,) + case.shape) + 1j * rng.standard_normal((3,) + case.shape)
        P = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps,
                      None, 0, ctx=vie_ctx)
        try:
            xd = torch.from_numpy(x).cuda()
            yd = torch.full_like(xd, complex("nan"))
            V.vie_matvec(P.handle, prec, 1e20 * xd, yd)
            V.vie_matvec(P.handle, prec, xd, yd)
            torch.cuda.synchronize()
            got = yd.cpu().numpy()
        finally:
            P.close()
        want = op.matvec_fft(g, x * g.mask)
        assert np.all(got[:, ~g.mask] == 0)
        err = np.abs(got - want).max() / np.abs(want).max()
        assert err <= TOL[prec], (shape, err)
