"""The far field's matrix form at the edges of its tiles: row tiles of 16
(z, y) rows, 32 mirror pairs of x per workgroup (odd and even nx, one pair to
several parts), direction tiles of 16 and blocks of 192, several row tiles per
workgroup.  Against the oracle's direct sum at the far field's tolerance
(1e-11: FP64 sums of up to 1e6 terms of order one, 1e-16 each)."""
import numpy as np
import pytest

import workloads as W
from oracle import operator as op, physics

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402


@pytest.mark.parametrize("shape,n_dir", [((1, 1, 1), 1), ((4, 4, 7), 16), ((3, 5, 8), 17), ((2, 9, 63), 49), ((5, 3, 64), 192),
                                         ((1, 17, 65), 193), ((4, 4, 129), 3), ((64, 130, 4), 5), ((96, 96, 130), 2)])
def test_far_field_tile_edges(vie_ctx, shape, n_dir):
    case = W.random_tiny(300 + shape[2], shape, fill=0.8, spacing=(0.04, 0.05, 0.03))
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(301)
    P = (rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)) * g.mask
    d = rng.standard_normal((n_dir, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    want = physics.far_field_vector(g, P, d)
    Pr = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                   ctx=vie_ctx)
    try:
        got = V.vie_far_field(Pr.handle, torch.from_numpy(P).cuda(), d)
    finally:
        Pr.close()
    assert np.linalg.norm(got - want) <= 1e-11 * np.linalg.norm(want)
