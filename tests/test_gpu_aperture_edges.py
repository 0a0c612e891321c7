"""Apertures at the ends of what the filter takes, in the kernels that form the
factors of their edges once: a point (D = 0), whose filter is 1, and an inner
diameter that is not positive (filled).  Every FP32-class kernel against FP64,
which evaluates the filter as it stands; within 1e-5 of the RMS (1e-3 in
split-BF16), as for any aperture.
"""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = {1: 1e-5, 2: 1e-3, 3: 1e-5, 4: 1e-5}


@pytest.fixture(scope="module")
def q():
    import paper_2404_02978_amd as q
    q.load_library()
    return q


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("precision", [1, 2, 3, 4])
@pytest.mark.parametrize("path,R,R_block", [(1, 6, 2), (1, 64, 64), (2, 64, 64)],
                         ids=["narrow", "fused", "two-phase"])
def test_edges(q, path, R, R_block, precision):
    K, P = 700, 40
    g = np.random.default_rng(4)
    D, d = g.uniform(0.5, 8.0, P), g.uniform(0.1, 0.4, P)
    D[::4], d[::4] = 0.0, 0.0
    d[1::4] = [0.0, -0.25, float("nan"), -0.0, -3.0] * 2
    with q.Context(0) as c:
        c.set_tuning(q.TUNE_WIDE_PATH, path)
        s = q.logpolar_sampler(1e-3, 1e2, index=5)
        fx, fy, area = c.sample_frequencies(s, math.ceil(R / R_block), K)
        w = c.weights(q.psd(0.1, 25.0), fx, fy, area)
        cx, cy = dev(g.uniform(-4, 4, P)), dev(g.uniform(-4, 4, P))
        print(f"path {path} R{R} Rb{R_block} p{precision}", flush=True)
        out, ref = (c.piston(K, fx, fy, w, cx, cy, dev(D), dev(d), R, R_block, rng=q.Rng(3, 7, 0),
                             precision=p).double() for p in (precision, 0))
        assert bool(torch.isfinite(ref).all())
        assert (out - ref).abs().max() <= TOL[precision] * ref.pow(2).mean().sqrt()
