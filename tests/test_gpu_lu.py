"""GPU shifted LU at the edges of its panels, tiles and window, against the
oracle's band LU: bandwidths at every change of the block size and of the
panel's rows per lane, orders around one block, ties and extreme scales of the
pivots.  Solutions within 1e-11 of the oracle's (complex128, condition
numbers up to 1e3) and the residual within 1e-13; a refined complex64 solve
meets its tolerance."""
import numpy as np
import pytest

import synth
from oracle import band as oband
from oracle import bandlu

pytestmark = pytest.mark.gpu


def _solve(ab, z, m, precision, seed):
    import torch
    import paper_2012_00506_amd as fb
    n = ab.shape[1]
    rng = np.random.default_rng(seed)
    Y = rng.standard_normal((n, m)) + 1j * rng.standard_normal((n, m))
    Yd = fb.to_colmajor(torch.from_numpy(Y))
    r = fb.band_shifted_solve(ab, z, [Yd] * len(z), precision=precision, ir_tol=1e-12, ir_max=8)
    return Y, r


def _check(ab, z, m, seed):
    Y, r = _solve(ab, z, m, 0, seed)
    for s, zz in enumerate(z):
        F = bandlu.shifted_band_lu(ab, zz)
        for got, ref in ((r.X[s], bandlu.lu_solve(F, Y)), (r.XH[s], bandlu.lu_solve_h(F, Y))):
            ref = np.asarray(ref)
            assert np.linalg.norm(got.cpu().numpy() - ref) <= 1e-11 * np.linalg.norm(ref)
    assert r.resid.max() <= 1e-13
    _, r1 = _solve(ab, z, m, 1, seed)
    assert r1.status == 0 and r1.resid.max() <= 1e-12


@pytest.mark.parametrize("b", [1, 15, 16, 17, 32, 33, 47, 48, 49, 56, 57, 64, 65, 80, 81, 96, 97,
                               112, 113, 120, 121, 128])
def test_lu_panel_and_tile_edges(b):
    print(f"lu edges b={b}", flush=True)
    for n in (b + 1, 2 * b + 9, 3 * b + 40):
        ab = synth.band_matrix(n, b, 31 * b + n, b % 2 == 0, -5, 5)
        _check(ab, np.array([0.3 + 0.7j, -1.1 - 0.4j]), 3, n)


@pytest.mark.parametrize("b", [8, 64, 100])
def test_lu_ties_and_zero_leading_pivots(b):
    """Entries of equal modulus (every search ties) and a zero diagonal, with a
    real shift off the spectrum's mean: interchanges in most columns."""
    n = 2 * b + 75
    rng = np.random.default_rng(b)
    ab = np.zeros((b + 1, n))
    for d in range(1, b + 1):
        ab[d, : n - d] = rng.choice([-1.0, 1.0], n - d)
    z = np.array([0.5 + 0.25j])
    dense = z[0] * np.eye(n) - oband.dense_from_band(ab)
    assert np.linalg.cond(dense) < 1e4
    _check(ab, z, 2, b)


@pytest.mark.parametrize("scale", [1e-120, 1e-25, 1e25, 1e120])
def test_lu_extreme_scales(scale):
    """Pivots whose squared modulus leaves the single (and, squared twice,
    approaches the double) range: the solution scales with the matrix."""
    import torch
    import paper_2012_00506_amd as fb
    n, b = 150, 20
    ab = synth.band_matrix(n, b, 5, True, -5, 5)
    z = 0.3 + 0.7j
    rng = np.random.default_rng(1)
    Y = rng.standard_normal((n, 2)) + 1j * rng.standard_normal((n, 2))
    Yd = fb.to_colmajor(torch.from_numpy(Y))
    ref = np.linalg.solve(z * np.eye(n) - oband.dense_from_band(ab), Y)
    r = fb.band_shifted_solve(ab * scale, [z * scale], [Yd], precision=0, resid=False)
    got = r.X[0].cpu().numpy() * scale
    assert np.linalg.norm(got - ref) <= 1e-11 * np.linalg.norm(ref)
