"""Band products and eigen residuals of one and four columns per thread: Ritz
values, vectors and residuals of rayleigh_ritz on both sides of the rule
(1024 workgroups), with column counts that leave 1, 2 and 3 columns in the last
group, a diagonal matrix and bands at the edges of a row block.  Bounds: those of
the Rayleigh-Ritz tests, the residuals recomputed with the oracle's band
product."""
import pytest

import synth
from test_gpu_rr import _block, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,m", [(2000, 5, 100), (2000, 5, 129), (2049, 0, 130), (2300, 31, 131),
                                   (20000, 3, 211)])
@pytest.mark.parametrize("cplx", [True, False])
def test_column_groups(n, b, m, cplx):
    import paper_2012_00506_amd as fb
    print(f"bandrows n={n} b={b} m={m} cplx={cplx}", flush=True)
    ab = synth.band_matrix(n, b, 60 + b, cplx, -20, 20)
    Q = _block(n, m, 900 + m, cplx, spread=1.0)
    [r] = fb.rayleigh_ritz(ab, [fb.to_colmajor(Q)])
    assert r.path == 0
    _check(ab, Q, r)
