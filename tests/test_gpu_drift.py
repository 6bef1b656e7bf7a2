"""Long runs keep their mass: FP32 against the same run in FP64 storage, FP64
against the method in 80-bit arithmetic (written here from Eq. 2, 3, 9 and 26 with
all non-flux rates 1).

A step rounds phi - phi_ref, of size a, by at most half a unit in the last place
of a, h = 2^(floor(log2 a) - 24) in FP32 and 2^(floor(log2 a) - 53) in FP64.  Rounding errors that change sign from step to
step grow like sqrt(n) h; errors of one sign, which a smooth or steady field
gives wherever sums are rounded at the size of phi in each step, grow like n h.
The bound is the first: sqrt(n) h, in the RMS over the nodes."""
import math

import numpy as np
import pytest

from paper_1603_09577_amd import workloads as W

pytestmark = pytest.mark.gpu


def _walls(ny, pw, source, rate=1.0):
    sp = W.spec_nonlinear_2d(64, ny, source=source)
    return dict(sp, s=[0.0] + [rate] * 8, bc=["periodic", "abb", "periodic"],
                phi_wall=[[0.0, 0.0], list(pw), [0.0, 0.0]]), W.noise_field((ny, 64), 3)


def _uniform(bcoef):
    return W.spec_nonlinear_2d(64, 48, bcoef=bcoef), np.full((48, 64), 0.5)


@pytest.mark.parametrize("spec,phi0", [_walls(200, (0.4, 0.6), False), _walls(90, (0.4, 0.6), True),
                                       _walls(90, (0.4, 0.6), False, 0.8), _uniform(0.5), _uniform(0.9)],
                         ids=["walls", "walls-source", "walls-0.8", "uniform-0.5", "uniform-0.9"])
def test_fp32_drift(spec, phi0):
    from paper_1603_09577_amd import lbm
    n = 4000
    a = lbm.Lbm(dict(spec, precision="f64")).init(phi0)
    b = lbm.Lbm(dict(spec, precision="f32")).init(phi0)
    a.step(n)
    b.step(n)
    ref = a.phi()
    size = float((ref - spec["phi_ref"]).abs().max())
    h = 2.0 ** (math.floor(math.log2(size)) - 24)
    rms = float((b.phi() - ref).pow(2).mean().sqrt())
    print(f"[gpu fp32 drift] rms {rms:.2e}, bound {math.sqrt(n) * h:.2e}", flush=True)
    assert rms <= math.sqrt(n) * h


def _extended(ny, source, pw, phi0, n):
    """phi after n steps of W.spec_nonlinear_2d, uniform in x, between walls."""
    L = np.longdouble
    sp = W.spec_nonlinear_2d(4, ny, source=source)
    b2, r = L(sp["b"][0][2]), [L(v) for v in sp["rpoly"]]
    kxx, kyy, kxy = L(sp["k0"][0][0]), L(sp["k0"][1][1]), L(sp["k0"][0][1])
    cx, cy = [0, 1, 0, -1, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1]
    w = [L(4) / 9] + [L(1) / 9] * 4 + [L(1) / 36] * 4

    def even(p, k):                                     # w_k (phi + 9/2 C : (c c - I/3)), C = int B' B'
        c = 4 * b2 * b2 * p ** 3 / 3
        return w[k] * (p + L(9) / 2 * (c * (cx[k] + cy[k]) ** 2 - 2 * c / 3))

    def level(p):                                       # A (Eq. 26), R and R (I - A / 2) B'
        k = 1 + p * p
        g = 3 * kxx * k + L(1) / 2, 3 * kyy * k + L(1) / 2, 3 * kxy * k
        det = g[0] * g[1] - g[2] ** 2
        a = g[1] / det, g[0] / det, -g[2] / det
        rr, bp = sum(c * p ** i for i, c in enumerate(r)) + 0 * p, 2 * b2 * p
        return a, rr, (rr * bp * (1 - (a[0] + a[2]) / 2), rr * bp * (1 - (a[2] + a[1]) / 2))

    phi = phi0.astype(L)
    g = [even(phi, k) + 3 * w[k] * (cx[k] + cy[k]) * b2 * phi * phi for k in range(9)]
    hist = phi
    for _ in range(n):
        phi = sum(g)
        a, rr, v = level(phi)
        _, rp, vp = level(hist)
        hist = phi
        se, b = L(3) / 2 * rr - rp / 2, b2 * phi * phi
        jx, jy = sum(c * x for c, x in zip(cx, g)) - b, sum(c * x for c, x in zip(cy, g)) - b
        d = ((a[0] - 1) * jx + a[2] * jy) / 6, (a[2] * jx + (a[1] - 1) * jy) / 6
        t = [3 * (b + L(3) / 2 * v[i] - vp[i] / 2) for i in range(2)]
        out = [even(phi, k) + w[k] * se + cx[k] * (w[k] * t[0] - d[0]) + cy[k] * (w[k] * t[1] - d[1]) for k in range(9)]
        g = [np.roll(out[k], cy[k]) for k in range(9)]
        for k, kb in ((2, 4), (5, 7), (6, 8)):
            g[k][0] = -out[kb][0] + 2 * even(L(pw[0]), k)
            g[kb][-1] = -out[k][-1] + 2 * even(L(pw[1]), kb)
    return sum(g)


@pytest.mark.skipif(np.finfo(np.longdouble).eps > 1e-18, reason="no 80-bit arithmetic")
@pytest.mark.parametrize("source", [False, True])
def test_fp64_drift(source):
    from paper_1603_09577_amd import lbm
    n, ny, pw = 4000, 90, (0.4, 0.6)
    phi0 = np.random.default_rng(1).uniform(0.4, 0.6, ny)
    spec = dict(W.spec_nonlinear_2d(4, ny, source=source), bc=["periodic", "abb", "periodic"],
                phi_wall=[[0.0, 0.0], list(pw), [0.0, 0.0]])
    s = lbm.Lbm(spec).init(np.repeat(phi0[:, None], 4, 1))
    s.step(n)
    ref = _extended(ny, source, pw, phi0, n)
    size = float(np.abs(ref - np.longdouble(spec["phi_ref"])).max())
    h = 2.0 ** (math.floor(math.log2(size)) - 53)
    rms = float(np.sqrt(np.mean((s.phi().cpu().numpy()[:, 0].astype(np.longdouble) - ref) ** 2)))
    print(f"[gpu fp64 drift] rms {rms:.2e}, bound {math.sqrt(n) * h:.2e}", flush=True)
    assert rms <= math.sqrt(n) * h
