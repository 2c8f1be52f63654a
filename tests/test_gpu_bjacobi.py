"""The Jacobi solvers of the reduced matrices around their limits (one
workgroup below 80 columns, a launch per round up to 256, blocks above), and
the pair problems of the parallel block Jacobi, real and complex: a reduced
matrix whose pairs are all real, all complex, or some of each (a basis on two
decoupled halves of the matrix, the first one real).  Oracle: LAPACK's
eigenvalues of the same reduced matrix.  Tolerance: two-sided Jacobi and LAPACK
are both backward stable, and the reduced matrix is formed twice (n eps
||B|| each), so the Ritz values agree to well within 1e-12 ||B||_1; the vectors
are orthonormal to m eps times a modest factor, below 1e-12."""
import numpy as np
import pytest

import synth
from oracle import band as oband

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["real", "complex", "mixed"])
@pytest.mark.parametrize("m", [79, 80, 81, 113, 255, 256, 257, 320, 385])
def test_pairs_real_and_complex(kind, m):
    import paper_2012_00506_amd as fb
    n, b, h = 900, 6, 450
    print(f"bjacobi kind={kind} m={m}", flush=True)
    ab = synth.band_matrix(n, b, 31, kind != "real", -20, 20)
    rng = np.random.default_rng(m)
    Q = rng.standard_normal((n, m))
    if kind != "real":
        Q = Q + 1j * rng.standard_normal((n, m))
    if kind == "mixed":
        ab[:, :h] = ab[:, :h].real
        for d in range(1, b + 1):
            ab[d, h - d:h] = 0.0  # the halves are decoupled
        k = m // 2
        Q[:h, :k] = Q[:h, :k].real
        Q[h:, :k] = 0.0
        Q[:h, k:] = 0.0
    Q, _ = np.linalg.qr(Q)
    r = fb.rayleigh_ritz(ab, [fb.to_colmajor(Q)])[0]
    A = Q.conj().T @ oband.dense_from_band(ab) @ Q
    lam = np.linalg.eigvalsh((A + A.conj().T) / 2)
    nrm = oband.norm1(ab)
    assert r.rank == m
    assert np.abs(np.sort(r.lam) - lam).max() <= 1e-12 * nrm
    X = r.X.cpu().numpy()
    assert np.abs(X.conj().T @ X - np.eye(m)).max() < 1e-12


@pytest.mark.parametrize("blocks", [1, 10, 20, 30])
@pytest.mark.parametrize("cplx", [True, False])
def test_shared_out_pairs(cplx, blocks):
    """A call with few pairs shares each pair's transformation out over 4 or 2
    workgroups and each tile of the update over 4 or 2, one with many does not:
    calls of 1, 10, 20 and 30 equal blocks (5, 50, 100 and 150 pairs; 40 tiles
    each), whose results are also equal to each other within a
    call.  (Between calls they differ by rounding: the Gram matrices' sums are
    split by the number of blocks.)"""
    import paper_2012_00506_amd as fb
    n, m = 400, 260
    print(f"bjacobi shared out cplx={cplx} blocks={blocks}", flush=True)
    ab = synth.band_matrix(n, 4, 33, cplx, -20, 20)
    rng = np.random.default_rng(5)
    Q = rng.standard_normal((n, m))
    if cplx:
        Q = Q + 1j * rng.standard_normal((n, m))
    Q, _ = np.linalg.qr(Q)
    out = fb.rayleigh_ritz(ab, [fb.to_colmajor(Q)] * blocks)
    A = Q.conj().T @ oband.dense_from_band(ab) @ Q
    lam = np.linalg.eigvalsh((A + A.conj().T) / 2)
    X = out[0].X.cpu().numpy()
    assert np.abs(np.sort(out[0].lam) - lam).max() <= 1e-12 * oband.norm1(ab)
    assert np.abs(X.conj().T @ X - np.eye(m)).max() < 1e-12
    for r in out[1:]:
        assert np.array_equal(r.lam, out[0].lam) and bool((r.X == out[0].X).all())
