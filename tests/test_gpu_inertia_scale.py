"""GPU inertia of matrices far from unit scale, at orders that the 16-column
panels do not divide: all three counts are the oracle's and do not change when
matrix and shifts are multiplied by 1e-30 .. 1e35, nor do shifts far beyond the
spectrum of an ordinary matrix (1e16 and more, where 1 + sigma rounds the 1
away) count rows that do not exist."""
import numpy as np
import pytest

import synth
from oracle import band as oband
from oracle import inertia as oin

pytestmark = pytest.mark.gpu


def _counts(ab, sh):
    import paper_2012_00506_amd as fb
    return [tuple(int(x) for x in v) for v in zip(*fb.band_inertia(ab, np.asarray(sh)))]


# below, at and above the order from which two halves are eliminated (2 b + 512)
@pytest.mark.parametrize("n,b", [(100, 8), (17, 1), (529, 8), (2 * 24 + 523, 24), (700, 113)])
@pytest.mark.parametrize("cplx", [False, True])
def test_counts_do_not_depend_on_the_scale(n, b, cplx):
    ab = synth.band_matrix(n, b, n + b, cplx, -6, 6)
    ev = np.linalg.eigvalsh(oband.dense_from_band(ab))
    sh = [0.5 * (ev[k - 1] + ev[k]) for k in (n // 5, n // 2)] + [ev[0] - 1.0, ev[-1] + 1.0]
    want = [(int((ev < s).sum()), 0, n - int((ev < s).sum())) for s in sh]
    for scale in (1.0, 1e-30, 1e16, 1e18, 1e35):
        print(f"inertia scale n={n} b={b} cplx={cplx} scale={scale}", flush=True)
        s = [scale * x for x in sh]
        assert [oin.inertia(scale * ab, x) for x in s] == want
        assert _counts(scale * ab, s) == want


@pytest.mark.parametrize("n,b", [(100, 8), (561, 24)])
@pytest.mark.parametrize("ns", [1, 130])
def test_shifts_far_beyond_the_spectrum(n, b, ns):
    ab = synth.band_matrix(n, b, 5, True, -6, 6)
    for s in (2.0**53, 1e16, 1e17, 3e25):
        print(f"inertia far shifts n={n} b={b} ns={ns} s={s}", flush=True)
        assert _counts(ab, [s] * ns) == [(n, 0, 0)] * ns
        assert _counts(ab, [-s] * ns) == [(0, 0, n)] * ns
