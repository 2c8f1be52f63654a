"""The two tile widths of the block solves: 16 and 32 right-hand sides per job
do the same operations in the same order for every column, so that a call's
solutions are equal bit for bit whichever width the sizes choose, and solve
the oracle's system to the residual bounds of the other solve tests (1e-13 in
complex128, ir_tol = 1e-12 refined).  Sizes: matrices smaller than a factor
block, a single block row, ragged last blocks and column tails of 1, 16 and
17 beyond a tile, and a call wide enough that the rule takes 32 columns."""
import numpy as np
import pytest

import synth
from oracle import bandlu as olu
from oracle import quadrature as oq

pytestmark = pytest.mark.gpu


def _solve(fb, ab, z, Y, precision):
    r = fb.band_shifted_solve(ab, z, [Y] * len(z), want_h=True, precision=precision,
                              ir_tol=1e-12, ir_max=6)
    assert r.status == 0
    return r


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,b,nsys,m", [(5, 4, 2, 33), (16, 15, 1, 1), (33, 32, 2, 17),
                                        (131, 64, 2, 48), (200, 40, 2, 49), (150, 20, 16, 250)])
def test_tile_widths_agree_bitwise(precision, n, b, nsys, m, tmp_path):
    import paper_2012_00506_amd as fb
    print(f"solve tiles precision={precision} n={n} b={b} nsys={nsys} m={m}", flush=True)
    ab = synth.band_matrix(n, b, 300 + n, True, -10, 10)
    z, _ = oq.contour(-1.0, 1.0, nsys)
    z = np.asarray(z)[:nsys]
    Yh = synth.rhs_block(n, m, n, True)
    Y = fb.to_colmajor(Yh)
    runs = [_solve(fb, ab, z, Y, precision)]  # the width that the rule chooses
    nb = (b + 15) // 16 * 16
    for v in (0, 2):
        path = tmp_path / f"tune{v}.json"
        path.write_text(f'{{"rsize": {4 if precision else 8}, "nb": {nb}, "variant": {v}}}\n')
        assert fb.tune_load(str(path)) == 1
        runs.append(_solve(fb, ab, z, Y, precision))
    for s in range(nsys):
        X = [r.X[s].cpu().numpy() for r in runs]
        XH = [r.XH[s].cpu().numpy() for r in runs]
        for q in (1, 2):
            assert np.array_equal(X[0], X[q]) and np.array_equal(XH[0], XH[q])
        tol = 1e-12 if precision else 1e-13
        assert olu.shifted_residual(ab, z[s], X[0], Yh).max() <= tol
        assert olu.shifted_residual(ab, z[s], XH[0], Yh, herm=True).max() <= tol
