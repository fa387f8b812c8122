"""z-pass variants at the z lengths 32 to 512, each of which has a geometry,
a choice to hold its twiddles and a choice to prefetch of its own: every
column-set variant (0, 2, 3, 4) against the oracle at the product's tolerance
(1e-12 in FP64, 1e-5 with FP32 transforms) and against variant 0 bit for bit,
which is what lets a rule on the column count pick among them without a solve's
steps depending on it.  Collocated and rooftop multiply; the mirror columns
(variant 1, collocated only) against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import operator as op, rooftop as rt

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2501_13512_amd import vie as V  # noqa: E402

TOL = {V.VIE_FP64: 1e-12, V.VIE_MIXED: 1e-5}
# (nz, ny, nx): z lengths 32, 36, 48, 64, 72, 96, 128, 144, 192, 256, 288, 384, 512
SHAPES = [(16, 5, 9), (18, 5, 6), (24, 6, 7), (32, 4, 9), (35, 6, 4), (48, 5, 5), (61, 4, 6), (70, 5, 7), (90, 4, 5),
          (128, 3, 5), (140, 4, 4), (180, 3, 6), (256, 3, 4)]


@pytest.mark.parametrize("rooftop", [False, True])
@pytest.mark.parametrize("prec", [V.VIE_FP64, V.VIE_MIXED])
@pytest.mark.parametrize("shape", SHAPES)
def test_column_variants(vie_ctx, shape, prec, rooftop):
    seed = 8000 + shape[0]
    if rooftop:   # one layer of vacuum on every side
        case = W.padded(W.random_tiny(seed, tuple(s - 2 for s in shape), fill=0.8))
    else:
        case = W.random_tiny(seed, shape, fill=0.8)
    assert case.shape == shape
    g = op.Grid.from_case(case)
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((3,) + shape) + 1j * rng.standard_normal((3,) + shape)
    want = rt.RooftopFFT(g)(x) if rooftop else op.FFTOperator(g)(x * g.mask)
    P = V.Problem(V.make_grid(case.nx, case.ny, case.nz, case.dx, case.dy, case.dz, case.wavelength), case.eps, None, 0,
                  ctx=vie_ctx, rooftop=rooftop)
    try:
        xd = torch.from_numpy(x).cuda()
        got = {}
        for v in (0, 2, 3, 4, -1) + (() if rooftop else (1,)):
            V.vie_problem_set_zpass(P.handle, prec, v)
            yd = torch.full_like(xd, complex("nan"))
            V.vie_matvec(P.handle, prec, xd, yd)
            torch.cuda.synchronize()
            got[v] = yd.cpu().numpy()
            assert np.abs(got[v] - want).max() <= TOL[prec] * np.abs(want).max(), v
    finally:
        P.close()
    for v in (2, 3, 4, -1):
        assert np.array_equal(got[v], got[0]), v
