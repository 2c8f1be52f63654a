"""Band products and eigen residuals by four columns per thread from the numbers
of workgroups that the rule asks for (16 and 1.5 per compute unit), with 1, 2 and 3
columns in the last group, and by one column below: Ritz values, vectors and
residuals against the oracle, with the bounds of the Rayleigh-Ritz tests."""
import pytest

import synth
from test_gpu_rr import _block, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,m", [(40000, 3, 153), (40000, 3, 154), (40000, 0, 155), (40000, 3, 100),
                                   (70000, 2, 1), (70000, 2, 3)])
@pytest.mark.parametrize("cplx", [True, False])
def test_column_groups(n, b, m, cplx):
    import paper_2012_00506_amd as fb
    print(f"bandcols n={n} b={b} m={m} cplx={cplx}", flush=True)
    ab = synth.band_matrix(n, b, 60 + b, cplx, -20, 20)
    Q = _block(n, m, 900 + m, cplx, spread=1.0)
    [r] = fb.rayleigh_ritz(ab, [fb.to_colmajor(Q)])
    assert r.path == 0
    _check(ab, Q, r)
