"""The work that users of this library have it do, as measurable cases.

Every case names a ``kind``: an entry point of ``paper_2012_00506_amd.api``
(or, for ``sample``, the three calls that make one training sample of the
slice planner) with the sizes, type and options of one call.  Matrices follow
the recipe of ``synth.band_matrix`` (linspace diagonal + N(0,1), sub-diagonals
N(0, 1/b)), drawn on the device from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2012_00506_amd import api

N_PLANNER = 80 * 256 + 256 + 256 * 256 + 256 + 256 * 64 + 64
NODES = 8


def listed():
    return [
        # count check of one slice of a small matrix: latency
        {"name": "inertia-small", "kind": "inertia", "n": 512, "b": 8, "cplx": False, "shifts": 2},
        # exact counts at the 17 boundaries of the 16 slices of the n=16384 b=64 workload
        {"name": "inertia-bounds", "kind": "inertia", "n": 16384, "b": 64, "cplx": True,
         "shifts": 17},
        # one training sample of the slice planner: features, Gershgorin bounds, 64 exact labels
        {"name": "planner-sample", "kind": "sample", "n": 12288, "b": 113, "cplx": False},
        # one optimiser step of the planner network at its training batch
        {"name": "planner-train", "kind": "train", "batch": 64},
        # equal-count slice placement before a solve
        {"name": "plan-equal-count", "kind": "plan", "n": 4096, "b": 48, "cplx": True, "K": 16},
        # a few shifted systems with a narrow block of right-hand sides, plain FP64, ragged
        {"name": "solve-f64-narrow", "kind": "solve", "n": 1000, "b": 30, "cplx": True,
         "systems": 4, "m": 24, "precision": 0},
        # one slice's nodes at a wide ragged band, complex64 refined to the FEAST default
        {"name": "solve-refined-b100", "kind": "solve", "n": 8191, "b": 100, "cplx": True,
         "systems": 8, "m": 200, "precision": 1},
        # a quarter of the n=16384 b=64 workload's filter sweep, complex64 + FP64 refinement
        {"name": "filter-refined-b64", "kind": "filter", "n": 16384, "b": 64, "cplx": True,
         "slices": 4, "width": 6.25, "m": 1450, "precision": 1},
        # the same sweep in plain FP64, on slices of uneven size
        {"name": "filter-f64-b64", "kind": "filter", "n": 16384, "b": 64, "cplx": True,
         "slices": 3, "width": 5.0, "m": 1111, "precision": 0},
        # the widest band, slices of the size that the n=65536 b=128 workload has
        {"name": "filter-refined-b128", "kind": "filter", "n": 16384, "b": 128, "cplx": True,
         "slices": 4, "width": 2.5, "m": 600, "precision": 1},
        # orthonormalisation and Rayleigh-Ritz of two slices' blocks
        {"name": "rayleigh-ritz", "kind": "rr", "n": 16384, "b": 64, "cplx": True, "blocks": 2,
         "m": 600},
        # a whole FEAST call: real n=2048 b=32, the 202 eigenvalues from -1 on (the slice
        # [-1, 1] of that workload), from random start vectors
        {"name": "feast-real-n2048", "kind": "feast", "n": 2048, "b": 32, "cplx": False,
         "range": 10.0, "lo": -1.0, "nev": 202},
    ]


def _logint(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(max(v, lo), hi)


def draw(rng):
    """One more case of the same ranges; sizes over their logarithm, odd ones
    among them, each kind bounded below its largest listed case's cost."""
    kind = rng.choice(["inertia", "inertia", "sample", "train", "plan", "solve", "solve", "filter",
                       "filter", "rr", "feast"])
    cplx = rng.random() < 0.6
    if kind == "inertia":
        b = _logint(rng, 1, 128)
        n = _logint(rng, max(256, 2 * b), 24576)
        return {"kind": kind, "n": n, "b": b, "cplx": cplx, "shifts": _logint(rng, 1, 128)}
    if kind == "sample":
        return {"kind": kind, "n": 256 * rng.randint(4, 48), "b": rng.randint(16, 128),
                "cplx": cplx}
    if kind == "train":
        return {"kind": kind, "batch": _logint(rng, 16, 512)}
    if kind == "plan":
        return {"kind": kind, "n": _logint(rng, 512, 6144), "b": _logint(rng, 4, 64), "cplx": cplx,
                "K": rng.randint(4, 32)}
    if kind == "solve":
        b = _logint(rng, 2, 128)
        return {"kind": kind, "n": _logint(rng, 400, 8192), "b": b, "cplx": cplx,
                "systems": _logint(rng, 1, 16), "m": _logint(rng, 1, 200),
                "precision": rng.randint(0, 1)}
    if kind == "filter":
        b = _logint(rng, 8, 128)
        return {"kind": kind, "n": _logint(rng, 1024, 16384), "b": b, "cplx": cplx,
                "slices": rng.randint(1, 4), "width": round(rng.uniform(2.0, 6.25), 2),
                "m": _logint(rng, 24, 600), "precision": rng.randint(0, 1)}
    if kind == "rr":
        return {"kind": kind, "n": _logint(rng, 2048, 16384), "b": _logint(rng, 8, 128),
                "cplx": cplx, "blocks": rng.randint(1, 3), "m": _logint(rng, 16, 500)}
    n = _logint(rng, 512, 2048)
    return {"kind": "feast", "n": n, "b": _logint(rng, 4, 48), "cplx": cplx, "range": 10.0,
            "lo": round(rng.uniform(-6.0, 4.0), 2), "nev": max(8, n * rng.randint(3, 9) // 100)}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, shape, cplx):
    re = torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    if not cplx:
        return re
    im = torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    return torch.complex(re, im) * math.sqrt(0.5)


def _band(c, g):
    """Row j of the (n, b+1) tensor holds B(j..j+b, j)."""
    n, b, half = c["n"], c["b"], c.get("range", 50.0)
    data = _randn(g, (n, b + 1), c["cplx"]) / math.sqrt(b)
    diag = torch.linspace(-half, half, n, dtype=torch.float64, device="cuda")
    data[:, 0] = (diag + torch.randn(n, generator=g, device="cuda",
                                     dtype=torch.float64)).to(data.dtype)
    rows = torch.arange(n, device="cuda")[:, None] + torch.arange(b + 1, device="cuda")[None, :]
    data[rows >= n] = 0
    return api.DeviceBand(n, b, c["cplx"], data)


def _block(g, n, m, cplx):
    return _randn(g, (m, n), cplx).t()


def _slices(c):
    """Adjacent slices of the given width, placed from -width * slices / 3 up."""
    lo = np.array([(i - c["slices"] / 3.0) * c["width"] for i in range(c["slices"])])
    return lo, lo + c["width"]


def _columns(c, i):
    """Columns of slice or block i: uneven, within 8 % below c["m"]."""
    return max(1, c["m"] - (i * 37) % max(1, c["m"] // 12 + 1))


def _shifts(c):
    """Shifts of the nodes of one slice after another (the upper half circles)."""
    z = []
    i = 0
    while len(z) < c["systems"]:
        zz, _ = api.contour_nodes(-3.0 + 1.5 * i, -1.5 + 1.5 * i, NODES)
        z += list(zz)
        i += 1
    return np.array(z[:c["systems"]])


def prepare(case, seed):
    c = dict(case)
    g = _gen(seed)
    s = {"c": c}
    if c["kind"] == "train":
        n = N_PLANNER
        s["w"] = torch.randn(n, generator=g, device="cuda") * 0.1
        s["opt"] = torch.cat([torch.randn(n, generator=g, device="cuda") * 1e-3,
                              torch.rand(n, generator=g, device="cuda") * 1e-4 + 1e-6])
        s["x"] = torch.randn((c["batch"], 80), generator=g, device="cuda")
        s["y"] = torch.sort(torch.rand((c["batch"], 64), generator=g, device="cuda"), dim=1)[0]
        return s
    B = s["B"] = _band(c, g)
    n, cplx = c["n"], c["cplx"]
    if c["kind"] == "inertia":
        r = np.random.default_rng(seed)
        s["shifts"] = np.sort(r.uniform(-50.0, 50.0, c["shifts"]))
    elif c["kind"] == "solve":
        s["z"] = _shifts(c)
        y = _block(g, n, c["m"], True)
        s["Y"] = [y] * c["systems"]  # the nodes of a slice share its block
    elif c["kind"] == "filter":
        lo, hi = _slices(c)
        m = [_columns(c, i) for i in range(c["slices"])]
        s["Y"] = [_block(g, n, mm, cplx) for mm in m]
        s["Q"] = [api.colmajor(n, mm, s["Y"][0].dtype) for mm in m]
        s["f"] = api.FeastFilter(B, lo, hi, m, n_nodes=NODES, precision=c["precision"],
                                 ir_tol=1e-12, ir_max=8)
    elif c["kind"] == "rr":
        # vectors as a warm start has them: each around its own row, where the
        # eigenvectors of a slice live
        rows = torch.arange(n, device="cuda", dtype=torch.float64)
        s["Q"] = []
        for i in range(c["blocks"]):
            m = _columns(c, i)
            at = (n - m) * (i + 1) / (c["blocks"] + 1) + torch.arange(m, device="cuda")
            env = torch.exp(-((rows[None, :] - at[:, None]) / 128.0) ** 2)
            s["Q"].append((_randn(g, (m, n), cplx) * env).t())
    elif c["kind"] == "feast":
        s["bounds"], s["counts"], _ = api.slice_plan(B, 1, "equal_count", lo=c["lo"],
                                                     nev=c["nev"])
        m = api.m0_rule(c["nev"])
        s["Y0"] = _block(g, n, m, cplx)
        s["Y"] = api.colmajor(n, m, s["Y0"].dtype)
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    c = s["c"]
    k = c["kind"]
    if k == "inertia":
        neg, zero, pos = api.band_inertia(s["B"], s["shifts"])
        return {"neg": neg, "zero": zero, "pos": pos}
    if k == "sample":
        x = api.band_features(s["B"], seed=7)
        _, ger = api.cheb_moments(s["B"], K=0, P=1, seed=7)
        sh = ger[0] + (np.arange(64) + 0.5) * (ger[1] - ger[0]) / 64
        neg, _, _ = api.band_inertia(s["B"], sh)
        return {"features": x, "gersh": ger, "neg": neg}
    if k == "train":
        loss = api.planner_train_step(s["w"], s["opt"], s["x"], s["y"], 1e-3, 10)
        return {"loss": loss, "w": s["w"], "opt": s["opt"]}
    if k == "plan":
        bounds, counts, evals = api.slice_plan(s["B"], c["K"], "equal_count")
        return {"bounds": bounds, "counts": counts, "evals": evals}
    if k == "solve":
        r = api.band_shifted_solve(s["B"], s["z"], s["Y"], want_h=True, precision=c["precision"],
                                   ir_tol=1e-12, ir_max=8, resid=False)
        return {"X": r.X, "XH": r.XH, "status": r.status}
    if k == "filter":
        r = s["f"](s["Y"], s["Q"])
        return {"Q": r.Q, "status": r.status}
    if k == "rr":
        res = api.rayleigh_ritz(s["B"], s["Q"])
        return {"lam": [r.lam for r in res], "X": [r.X for r in res], "rank": [r.rank for r in res]}
    s["Y"].copy_(s["Y0"])
    r = api.feast_band_slice(s["B"], s["bounds"][:1], s["bounds"][1:], [s["Y"]],
                             m_expected=s["counts"])[0]
    return {"lam": r.lam, "X": r.X, "m": r.m_found, "info": r.info, "iters": r.iters}


# ------------------------------------------------------------------ work

def work(case):
    """Bytes: each input and output once.  Flops: the factorisations, solves
    and products of one pass (complex arithmetic: 8 per multiply-add)."""
    c = case
    k = c["kind"]
    if k == "train":
        rows = c["batch"]
        macs = 80 * 256 + 256 * 256 + 256 * 64
        return {"bytes": 4.0 * (6 * N_PLANNER + rows * 144), "flops": 6.0 * rows * macs}
    n, b = c["n"], c["b"]
    el, f = (16.0, 8.0) if c["cplx"] else (8.0, 2.0)
    band = el * n * (b + 1)
    if k == "inertia":
        return {"bytes": band + 20.0 * c["shifts"], "flops": f / 2 * n * b * b * c["shifts"]}
    if k == "sample":
        return {"bytes": band, "flops": f / 2 * n * b * b * 64 + 16 * 20 * f * n * (2 * b + 1)}
    if k == "plan":  # about log2 of the boundaries' resolution, six rounds, two certificates
        return {"bytes": band, "flops": f / 2 * n * b * b * 8 * c["K"]}
    lu, col = 16.0 * n * b * b, 24.0 * n * b
    if k == "solve":
        return {"bytes": band + 16.0 * n * c["m"] * (1 + 2 * c["systems"]),
                "flops": c["systems"] * (lu + 2 * c["m"] * col)}
    if k == "filter":
        m = sum(_columns(c, i) for i in range(c["slices"]))
        dirs = 2 if c["cplx"] else 1
        return {"bytes": band + 2 * el * n * m,
                "flops": NODES * (c["slices"] * lu + dirs * m * col)}
    if k == "rr":
        m = [_columns(c, i) for i in range(c["blocks"])]
        return {"bytes": band + 2 * el * n * sum(m),
                "flops": sum(f * (2.5 * n * v * v + n * (2 * b + 1) * v) + 3 * f * v ** 3
                             for v in m)}
    m, its, dirs = max(1.5 * c["nev"], c["nev"] + 10), 3, 2 if c["cplx"] else 1
    return {"bytes": band + 2 * el * n * m,
            "flops": its * (NODES * (lu + dirs * m * col) + f * 2.5 * n * m * m + 3 * f * m ** 3)}


# ------------------------------------------------------------------ 64 bits

def _solve_cost(n, b, systems, m):
    return systems * 8.0 * n * b * (4.0 * b + 5.0 * m)


def _blocks(B):
    """Diagonal and lower blocks (order p, b rounded up) of the band, host."""
    n, b = B.n, B.b
    p = min(max(b, 16), n)
    K = -(-n // p)
    ab = B.data.cpu().numpy()
    D = np.zeros((K, p, p), np.complex128)
    L = np.zeros((K, p, p), np.complex128)  # L[k] = B(block k, block k - 1)
    for d in range(b + 1):
        j = np.arange(n - d)
        i = j + d
        same = i // p == j // p
        v = ab[j, d]
        D[i[same] // p, i[same] % p, j[same] % p] = v[same]
        D[i[same] // p, j[same] % p, i[same] % p] = np.conj(v[same])
        o = ~same
        L[i[o] // p, i[o] % p, j[o] % p] = v[o]
    idx = np.arange(p)
    D[:, idx, idx] = D[:, idx, idx].real
    return D, L, p, K


def _solver(blocks, n, z):
    """Solver of (z I - B) x = y by block elimination (z off the real axis)."""
    D, L, p, K = blocks
    last = n - (K - 1) * p
    eye = np.eye(p)
    inv, S = [], None
    for k in range(K):
        S = z * eye - D[k]
        if k == K - 1 and last < p:  # identity beyond n
            S[last:, :] = 0
            S[:, last:] = 0
            S[np.arange(last, p), np.arange(last, p)] = 1
        if k:
            S = S - L[k] @ (inv[k - 1] @ np.conj(L[k].T))
        inv.append(np.linalg.inv(S))

    def solve(Y):
        m = Y.shape[1]
        y = np.zeros((K * p, m), np.complex128)
        y[:n] = Y
        y = y.reshape(K, p, m)
        for k in range(1, K):
            y[k] += L[k] @ (inv[k - 1] @ y[k - 1])
        y[K - 1] = inv[K - 1] @ y[K - 1]
        for k in range(K - 2, -1, -1):
            y[k] = inv[k] @ (y[k] + np.conj(L[k + 1].T) @ y[k + 1])
        return y.reshape(K * p, m)[:n]
    return solve


def _dense(B):
    n, b = B.n, B.b
    ab = B.data.cpu().numpy()
    A = np.zeros((n, n), ab.dtype)
    for d in range(b + 1):
        j = np.arange(n - d)
        A[j + d, j] = ab[j, d]
        A[j, j + d] = np.conj(ab[j, d])
    return A


def exact(case, seed):
    c = case
    k = c["kind"]
    if k == "solve":
        if 2 * _solve_cost(c["n"], c["b"], c["systems"], c["m"]) > 3e11:
            return None
        s = prepare(c, seed)
        blocks = _blocks(s["B"])
        Y = s["Y"][0].cpu().numpy()
        # B is Hermitian: the conjugate-transposed system is the one at conj(z)
        return {"X": [_solver(blocks, c["n"], z)(Y) for z in s["z"]],
                "XH": [_solver(blocks, c["n"], np.conj(z))(Y) for z in s["z"]], "status": None}
    if k == "filter":
        if 2 * _solve_cost(c["n"], c["b"], NODES * c["slices"], c["m"]) > 3e11:
            return None
        s = prepare(c, seed)
        blocks = _blocks(s["B"])
        lo, hi = _slices(c)
        out = []
        x, wt = np.polynomial.legendre.leggauss(NODES)
        for i in range(c["slices"]):
            Y = s["Y"][i].cpu().numpy()
            mid, r = (lo[i] + hi[i]) / 2, (hi[i] - lo[i]) / 2
            Q = np.zeros(Y.shape, np.complex128)
            for t, w in zip(x, wt):
                e = np.exp(1j * math.pi / 2 * (1 - t))
                z, a = mid + r * e, w / 4 * r * e
                Q += a * _solver(blocks, c["n"], z)(Y)
                if c["cplx"]:
                    Q += np.conj(a) * _solver(blocks, c["n"], np.conj(z))(Y)
            out.append(Q if c["cplx"] else 2 * Q.real)
        return {"Q": out, "status": None}
    if k == "rr":
        m = [_columns(c, i) for i in range(c["blocks"])]
        if max(m) > 700 or c["n"] * max(m) ** 2 * 8.0 * len(m) > 2e11:
            return None
        s = prepare(c, seed)
        ab = s["B"].data.cpu().numpy()
        lam = []
        for q in s["Q"]:
            q = np.linalg.qr(q.cpu().numpy())[0]
            bq = ab[:, :1].real * q
            for d in range(1, c["b"] + 1):
                v = ab[:c["n"] - d, d][:, None]
                bq[d:] += v * q[:-d]
                bq[:-d] += np.conj(v) * q[d:]
            lam.append(np.linalg.eigvalsh(np.conj(q.T) @ bq))
        return {"lam": lam, "X": [None] * len(lam), "rank": [None] * len(lam)}
    if k == "feast":
        s = prepare(c, seed)
        lam = np.linalg.eigvalsh(_dense(s["B"]))
        lam = lam[(lam >= s["bounds"][0]) & (lam < s["bounds"][1])]
        return {"lam": lam, "X": None, "m": None, "info": None, "iters": None}
    return None  # whole numbers, or features and weights without a plain 64-bit form
