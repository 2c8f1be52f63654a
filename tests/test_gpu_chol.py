"""The diagonal blocks of the Cholesky QR: block sizes of 1, 2, 63, 64 and the
first sizes beyond one and two blocks, and a pivot that fails in the first,
an inner and the last column of a block or of its 4 x 4 register tiles.
Full-rank blocks take the Cholesky path and give the oracle's Ritz values to
1e-12 ||B||_1 and orthonormal vectors to 1e-12 (the bounds of the
Rayleigh-Ritz tests); a column equal to another one makes its pivot zero, so
that the block takes the eigen path with one column less."""
import numpy as np
import pytest

import synth
from test_gpu_rr import _block, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx", [True, False])
def test_block_sizes(cplx):
    import paper_2012_00506_amd as fb
    ab = synth.band_matrix(500, 8, 51, cplx, -20, 20)
    ms = [1, 2, 3, 4, 5, 63, 64, 65, 66, 127, 128, 129]
    Qs = [_block(500, m, 700 + m, cplx, spread=2.0) for m in ms]
    print(f"chol cplx={cplx} ms={ms}", flush=True)
    for q, r in zip(Qs, fb.rayleigh_ritz(ab, [fb.to_colmajor(q) for q in Qs])):
        assert r.path == 0
        _check(ab, q, r)


@pytest.mark.parametrize("m,col", [(2, 1), (10, 3), (64, 63), (66, 64), (70, 36), (129, 128)])
def test_failed_pivot(m, col):
    import paper_2012_00506_amd as fb
    ab = synth.band_matrix(500, 8, 52, True, -20, 20)
    Q = _block(500, m, 800 + m, True)
    Q[:, col] = Q[:, 0]
    print(f"chol failed pivot m={m} col={col}", flush=True)
    r = fb.rayleigh_ritz(ab, [fb.to_colmajor(Q)])[0]
    assert r.path == 1 and r.rank == m - 1
    X = r.X[:, : r.rank].cpu().numpy()
    assert np.abs(X.conj().T @ X - np.eye(r.rank)).max() < 1e-12
