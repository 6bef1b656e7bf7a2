"""Long FP32 runs keep their mass: phi against the same run in FP64 storage.

A step rounds phi - phi_ref, of size a, by at most half a unit in the last place
of a, h = 2^(floor(log2 a) - 24).  Rounding errors that change sign from step to
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
