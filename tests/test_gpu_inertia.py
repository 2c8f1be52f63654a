"""GPU inertia at the edges of its tiles and of its split elimination, against
the oracle's unblocked band LDL^H: counts are whole numbers and equal wherever
the shift is farther than 1e-8 ||B||_1 from every eigenvalue (checked with
LAPACK), and zero pivots that no other row couples to are counted alike."""
import numpy as np
import pytest

import synth
from oracle import band as oband
from oracle import inertia as oin

pytestmark = pytest.mark.gpu


def _shifts(ab, k, seed):
    ev = np.linalg.eigvalsh(oband.dense_from_band(ab))
    delta = 1e-8 * oband.norm1(ab)
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < k:
        s = rng.uniform(ev[0] - 1, ev[-1] + 1)
        if np.min(np.abs(ev - s)) > delta:
            out.append(s)
    return np.array(out), ev


# window tiles change at b = 1, 17, 33, ..; the halves start at n = 2 b + 512
@pytest.mark.parametrize("b", [1, 2, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113,
                               127, 128])
@pytest.mark.parametrize("cplx", [False, True])
def test_tile_edges_whole_and_split(b, cplx):
    import paper_2012_00506_amd as fb
    for n in (b + 1, 2 * b + 17, 2 * b + 511, 2 * b + 512, 2 * b + 529):
        print(f"inertia edges n={n} b={b} cplx={cplx}", flush=True)
        ab = synth.band_matrix(n, b, 7 * n + b, cplx, -6, 6)
        sh, ev = _shifts(ab, 3, n)
        neg, zero, pos = fb.band_inertia(ab, sh)
        assert list(neg) == [int((ev < s).sum()) for s in sh]
        assert not zero.any() and np.all(neg + pos == n)


@pytest.mark.parametrize("ns", [1, 128, 129, 300])
def test_shift_counts_around_the_split_limit(ns):
    import paper_2012_00506_amd as fb
    ab = synth.band_matrix(900, 20, 3, True, -8, 8)
    sh, ev = _shifts(ab, ns, ns)
    neg, _, _ = fb.band_inertia(ab, sh)
    assert list(neg) == [int((ev < s).sum()) for s in sh]


@pytest.mark.parametrize("rows", [[0], [3, 50], [399], [400, 401], [640, 798], [10, 420, 790]])
@pytest.mark.parametrize("cplx", [False, True])
def test_zero_pivots_in_either_half_and_the_separator(rows, cplx):
    import paper_2012_00506_amd as fb
    n, b = 800, 24
    ab = synth.band_matrix(n, b, 11, cplx, -6, 6)
    for r in rows:  # row r decoupled, its diagonal on the shift
        ab[0, r] = 0.25
        ab[1:, r] = 0
        for d in range(1, min(b, r) + 1):
            ab[d, r - d] = 0
    for sh in ([0.25], [0.25, -1.5]):
        neg, zero, pos = fb.band_inertia(ab, sh)
        got = [tuple(int(x) for x in v) for v in zip(neg, zero, pos)]
        assert got == [oin.inertia(ab, s) for s in sh]
        assert zero[0] == len(rows)
