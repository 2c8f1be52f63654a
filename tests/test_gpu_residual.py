"""The FP64 residuals of the shifted solves for every factor block size, ragged
last blocks and column tails: band_shifted_solve with a loose ir_tol returns
the plain complex64 solutions and the largest residual ratio of each system,
which the oracle recomputes from the same solutions.  A complex64 residual is
about 1e-7 ||A|| ||x||, and both sides round at (2 b + 1) eps ||A|| ||x|| at
most, 3e-14 of it for b = 128: the ratios agree to 1e-6 relative."""
import numpy as np
import pytest

import synth
from oracle import bandlu as olu
from oracle import quadrature as oq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,m", [(7, 3, 1), (300, 16, 17), (97, 32, 33), (200, 44, 31),
                                   (640, 64, 49), (333, 70, 16), (300, 96, 5), (500, 101, 19),
                                   (129, 128, 15), (700, 128, 32)])
def test_residual_ratio(n, b, m):
    import paper_2012_00506_amd as fb
    print(f"residual n={n} b={b} m={m}", flush=True)
    ab = synth.band_matrix(n, b, 400 + n, True, -10, 10)
    z, _ = oq.contour(-1.0, 1.0, 8)
    z = np.asarray(z)[[0, 5]]
    Yh = synth.rhs_block(n, m, n, True)
    r = fb.band_shifted_solve(ab, z, [fb.to_colmajor(Yh)] * 2, want_h=True, precision=1,
                              ir_tol=1e-2, ir_max=6)
    assert r.status == 0 and r.passes.max() == 0
    for s in range(2):
        ref = max(olu.shifted_residual(ab, z[s], r.X[s].cpu().numpy(), Yh).max(),
                  olu.shifted_residual(ab, z[s], r.XH[s].cpu().numpy(), Yh, herm=True).max())
        assert abs(r.resid[s] - ref) <= 1e-6 * ref, (s, r.resid[s], ref)
