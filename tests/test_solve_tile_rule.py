"""The tile width of the block solves: the rule on the size of a call (complex64
calls with a 32-column tile per compute unit or more take 32 columns, all others
16), the choices that tune files hold, and, on the GPU, calls on both sides of
the line against the forced widths, which do the same operations in the same
order for every column, so that solutions are equal bit for bit."""
import ctypes as C

import numpy as np
import pytest

import synth
from oracle import quadrature as oq


def _lib():
    from paper_2012_00506_amd import _native as N
    return N.lib()


def _tile(precision, b, tiles32):
    L = _lib()
    f = L._ZN2fb10solve_tileIfEEiim if precision else L._ZN2fb10solve_tileIdEEiim
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_size_t]
    return f(b, tiles32)


def _tune(tmp_path, precision, nb, v):
    path = tmp_path / f"tune{v}.json"
    path.write_text(f'{{"rsize": {4 if precision else 8}, "nb": {nb}, "variant": {v}}}\n')
    assert _lib().fb_tune_load(str(path).encode()) == 1


@pytest.mark.parametrize("b", [1, 16, 20, 48, 64, 65, 128])
def test_rule(b):
    for tiles in (0, 1, 255, 256, 100000):
        assert _tile(1, b, tiles) == (32 if tiles >= 256 and b <= 64 else 16)
        assert _tile(0, b, tiles) == 16


@pytest.mark.parametrize("precision", [0, 1])
def test_every_number_of_a_tune_file_is_a_kernel(precision, tmp_path):
    for v in range(10):
        wide = 2 <= v < 6 or v == 9
        for nb in (16, 64, 80, 128):
            _tune(tmp_path, precision, nb, v)
            for tiles in (1, 256):
                # blocks above 64 rows have the narrow kernel only
                assert _tile(precision, nb, tiles) == (32 if wide and nb <= 64 else 16)


@pytest.mark.parametrize("precision", [0, 1])
def test_workspace_does_not_depend_on_the_tuned_width(precision, tmp_path):
    from paper_2012_00506_amd import _native as N
    n, b, m = 5000, 40, 70

    def size():
        bs = N.fb_band(n, b, 2, b + 1, C.c_void_p(1))
        P, ld, lw = (C.c_void_p * 1)(1), (C.c_int64 * 1)(n), C.c_size_t(0)
        o = N.fb_solve_opts(precision, 1e-10, 4, 0)
        assert _lib().band_shifted_solve(C.byref(bs), 1, (C.c_double * 2)(0.1, 0.2),
                                         (C.c_int32 * 1)(m), P, ld, P, P, ld, (C.c_double * 1)(),
                                         None, C.byref(o), None, C.byref(lw), None) == 0
        return lw.value

    sizes = {size()}
    for v in (0, 2):
        _tune(tmp_path, precision, 48, v)
        sizes.add(size())
    assert len(sizes) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,b,m", [(150, 20, 256), (150, 20, 224), (131, 64, 250), (70, 16, 241)])
def test_rule_and_forced_widths_agree_bitwise(n, b, m, precision, tmp_path):
    import paper_2012_00506_amd as fb
    nsys, nb = 16, (b + 15) // 16 * 16
    tiles = 2 * nsys * ((m + 31) // 32)
    print(f"tile rule precision={precision} n={n} b={b} m={m} tiles={tiles}", flush=True)
    assert _tile(precision, b, tiles) == (32 if precision and tiles >= 256 else 16)
    ab = synth.band_matrix(n, b, 300 + n, True, -10, 10)
    z = np.asarray(oq.contour(-1.0, 1.0, nsys)[0])[:nsys]
    Y = [fb.to_colmajor(synth.rhs_block(n, m, n, True))] * nsys
    runs = []
    for v in (None, 0, 2):
        if v is not None:
            _tune(tmp_path, precision, nb, v)
            assert _tile(precision, b, tiles) == (32 if v else 16)
        r = fb.band_shifted_solve(ab, z, Y, want_h=True, precision=precision, ir_tol=1e-12,
                                  ir_max=6)
        assert r.status == 0
        runs.append(r)
    for r in runs[1:]:
        for s in range(nsys):
            assert bool((r.X[s] == runs[0].X[s]).all()) and bool((r.XH[s] == runs[0].XH[s]).all())
