"""The scratch of split eliminations is asked for by workspace queries and can
be left out: at n = 767 it begins at b = 127 (n >= 2 b + 512), and a workspace
sized for b = 128, which is larger in everything else, serves b = 127 with the
same results."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

N_, RANGE = 767, 20


def _inertia(fb, B, ab, ev):
    return list(fb.band_inertia(B, np.linspace(-25, 25, 9)))


def _certify(fb, B, ab, ev):
    return list(fb.slice_certify(B, np.linspace(-25, 25, 5)))


def _plan(fb, B, ab, ev):
    return list(fb.slice_plan(B, 4, mode="equal_width", lo=-25, hi=25))


def _plan_prev(fb, B, ab, ev):
    return list(fb.slice_plan_prev(B, ev, 100, 4))


def _feast(fb, B, ab, ev):
    lo, hi = 0.5 * (ev[300] + ev[301]), 0.5 * (ev[320] + ev[321])
    Y = [fb.to_colmajor(synth.rhs_block(N_, 32, 7, True))]
    r = fb.feast_band_slice(B, [lo], [hi], Y, tol=1e-9, max_iter=20)[0]
    assert r.m_found == 20 and r.info == 0
    return [r.m_found, r.evals]


@pytest.mark.parametrize("call", [_inertia, _certify, _plan, _plan_prev, _feast])
def test_workspace_of_the_wider_band_serves_the_narrower(call, monkeypatch):
    import torch
    import paper_2012_00506_amd as fb
    from paper_2012_00506_amd import api
    sizes, cap = [], [None]

    def workspace(_, lw, device):
        sizes.append(int(lw.value))
        size = sizes[-1] if cap[0] is None else min(sizes[-1], cap[0])
        return torch.empty(max(size, 256), dtype=torch.uint8, device=device)

    monkeypatch.setattr(api, "_workspace", workspace)
    out = []
    for b, limit in ((128, None), (127, None), (127, 0)):
        cap[0] = limit if limit is None else sizes[0]
        print(f"inertia workspace {call.__name__} b={b} cap={cap[0]}", flush=True)
        ab = synth.band_matrix(N_, b, 3, True, -RANGE, RANGE)
        ev = np.linalg.eigvalsh(_dense(ab))
        out.append(call(fb, fb.DeviceBand.from_band(ab), ab, ev))
    assert sizes[1] > sizes[0]  # the scratch is asked for
    for a, b in zip(out[1], out[2]):
        assert np.array_equal(np.asarray(a), np.asarray(b))


def _dense(ab):
    from oracle import band as oband
    return oband.dense_from_band(ab)
