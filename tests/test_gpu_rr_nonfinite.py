"""Rayleigh-Ritz of a block that holds a NaN or an infinity: no direction of it is
kept (rank 0) and the blocks beside it are solved as ever.  Sizes of the three
Jacobi solvers, whose eigenvalues are then NaN and have to be ranked all the
same: the ranks index the vectors."""
import numpy as np
import pytest

import synth
from oracle import band as oband

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [40, 100, 300])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("cplx", [True, False])
def test_nonfinite_block_is_dropped(m, value, cplx):
    import paper_2012_00506_amd as fb
    n = 400
    print(f"rr nonfinite m={m} value={value} cplx={cplx}", flush=True)
    ab = synth.band_matrix(n, 4, 9, cplx, -20, 20)
    rng = np.random.default_rng(m)
    Q = rng.standard_normal((n, m))
    if cplx:
        Q = Q + 1j * rng.standard_normal((n, m))
    Q, _ = np.linalg.qr(Q)
    bad = Q.copy()
    bad[7, m // 2] = value
    r = fb.rayleigh_ritz(ab, [fb.to_colmajor(bad), fb.to_colmajor(Q)])
    A = Q.conj().T @ oband.dense_from_band(ab) @ Q
    lam = np.linalg.eigvalsh((A + A.conj().T) / 2)
    assert r[0].rank == 0
    assert r[1].rank == m and np.abs(r[1].lam - lam).max() <= 1e-12 * oband.norm1(ab)
