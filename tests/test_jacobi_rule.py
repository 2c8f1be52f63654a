"""The rule that chooses between one workgroup per reduced matrix and a launch
per round of the cyclic Jacobi: both sides of its line at sizes and numbers of
matrices that were measured (host-only), and, on the GPU, calls on both sides
against LAPACK.  Tolerances as in the block Jacobi tests: 1e-12 ||B||_1 for the
Ritz values, 1e-12 for the vectors' orthonormality."""
import ctypes as C

import numpy as np
import pytest

import synth
from oracle import band as oband


def _rounds(ms, cus=256):
    from paper_2012_00506_amd import _native as N
    f = N.lib()._ZN2fb10rounds_payEili
    f.restype, f.argtypes = C.c_bool, [C.c_int, C.c_int64, C.c_int]
    return f(max(ms), sum(m * m for m in ms), cus)


@pytest.mark.parametrize("ms", [[80], [80] * 8, [96] * 16, [128] * 32, [160] * 32, [200] * 64,
                                [250] * 32, [80] + [20] * 128, [250] + [79] * 128])
def test_rounds_where_they_are_faster(ms):
    assert _rounds(ms)


@pytest.mark.parametrize("ms", [[79], [20] * 9, [80] * 16, [80] * 128, [96] * 64, [128] * 64,
                                [128] * 128, [160] * 128, [200] * 128])
def test_one_workgroup_each_where_that_is_faster(ms):
    assert not _rounds(ms)


def test_fewer_compute_units_take_fewer_matrices_by_rounds():
    assert _rounds([128] * 40, cus=256) and not _rounds([128] * 40, cus=64)


@pytest.mark.gpu
@pytest.mark.parametrize("m,blocks", [(80, 9), (80, 10), (97, 32), (97, 33), (255, 75)])
@pytest.mark.parametrize("cplx", [True, False])
def test_both_sides_against_lapack(m, blocks, cplx):
    import paper_2012_00506_amd as fb
    n = max(200, m + 13)
    print(f"jacobi rule m={m} blocks={blocks} cplx={cplx}", flush=True)
    ab = synth.band_matrix(n, 4, 33, cplx, -20, 20)
    rng = np.random.default_rng(m)
    Q = rng.standard_normal((n, m))
    if cplx:
        Q = Q + 1j * rng.standard_normal((n, m))
    Q, _ = np.linalg.qr(Q)
    out = fb.rayleigh_ritz(ab, [fb.to_colmajor(Q)] * blocks)
    A = Q.conj().T @ oband.dense_from_band(ab) @ Q
    lam = np.linalg.eigvalsh((A + A.conj().T) / 2)
    X = out[0].X.cpu().numpy()
    assert out[0].rank == m
    assert np.abs(out[0].lam - lam).max() <= 1e-12 * oband.norm1(ab)
    assert np.abs(X.conj().T @ X - np.eye(m)).max() < 1e-12
    for r in out[1:]:
        assert np.array_equal(r.lam, out[0].lam) and bool((r.X == out[0].X).all())
