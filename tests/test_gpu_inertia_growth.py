"""GPU inertia where one of the two elimination directions meets pivots near
rounding level: rows at an end of the band whose own diagonal block is noise
(an augmented system with a zero block).  Eliminated towards those rows the
factorisation is harmless, away from them its elements grow and their digits
are lost; counts have to be those of the plain order, leading rows first, which
is the oracle's, wherever that one counts what LAPACK finds."""
import numpy as np
import pytest

import synth
from oracle import band as oband
from oracle import inertia as oin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 8, 12])
@pytest.mark.parametrize("noise", [1e-25, 3e-17, 1e-12, 1e-9])
@pytest.mark.parametrize("cplx", [False, True])
def test_trailing_rows_with_a_diagonal_block_of_noise(rows, noise, cplx):
    import paper_2012_00506_amd as fb
    n, b = 700, 24
    bad = []
    for seed in range(8):
        print(f"inertia growth rows={rows} noise={noise} cplx={cplx} seed={seed}", flush=True)
        ab = synth.band_matrix(n, b, seed, cplx, -6, 6)
        ab[:, n - rows:] = 0
        ab[0, n - rows:] = noise * np.random.default_rng(seed).standard_normal(rows)
        ev = np.linalg.eigvalsh(oband.dense_from_band(ab))
        sh = [s for s in (0.0, 0.5, -1.25) if np.min(np.abs(ev - s)) > 1e-8 * oband.norm1(ab)]
        want = [(int((ev < s).sum()), 0, n - int((ev < s).sum())) for s in sh]
        assert sh and [oin.inertia(ab, s) for s in sh] == want
        got = [tuple(int(x) for x in v) for v in zip(*fb.band_inertia(ab, np.array(sh)))]
        if got != want:
            bad.append((seed, got, want))
    assert not bad
