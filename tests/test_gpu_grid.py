"""Fields of narrow frequency sets on regular grids, which are found on the
device from the points and summed through their product structure, against
the FP64 oracle: both orders of the points, ragged and extreme shapes, points
that are almost a grid, and the calls whose points are none.

Tolerances relative to the RMS of the oracle's field: 1e-11 (FP64), 1e-5
(FP32 class), as for the general kernels.
"""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TOL = {0: 1e-11, 1: 1e-5, 2: 1e-5, 4: 1e-5}


@pytest.fixture(scope="module")
def q():
    import paper_2404_02978_amd as q
    q.load_library()
    return q


@pytest.fixture(scope="module")
def ctx(q):
    c = q.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.double().cpu().numpy()


def grid(ny, nx, order, seed=0):
    """Unevenly spaced coordinates: only the product structure matters."""
    rng = np.random.default_rng([ny, nx, seed])
    x, y = np.sort(rng.uniform(-3, 3, nx)), np.sort(rng.uniform(-3, 3, ny))
    if order == "x":
        return np.tile(x, ny), np.repeat(y, nx)
    return np.repeat(x, ny), np.tile(y, nx)


def run(q, ctx, px, py, K, R, R_block, precision, mode=0, coef=None, name=""):
    s = q.logpolar_sampler(1e-3, 1e2, index=9)
    fx, fy, area = ctx.sample_frequencies(s, math.ceil(R / R_block), K)
    w = ctx.weights(q.psd(0.1, 25.0), fx, fy, area)
    print(f"{name} P{px.size} K{K} R{R} Rb{R_block} p{precision} mode{mode}", flush=True)
    kw = dict(coef=dev(coef)) if coef is not None else dict(rng=q.Rng(6, 21, mode))
    out = ctx.synthesize_phase(K, fx, fy, w, dev(px), dev(py), R, R_block, precision=precision,
                               **kw)
    ref = oracle.synthesize(host(fx), host(fy), host(w), px, py, R, R_block, K=K, seed=6,
                            counter=21, mode=mode, coef=coef)
    e = np.max(np.abs(host(out) - ref)) / math.sqrt(np.mean(ref * ref))
    print(f"  eps_max {e:.2e}", flush=True)
    assert e <= TOL[precision]


@pytest.mark.parametrize("precision", [0, 1, 4])
@pytest.mark.parametrize("order", ["x", "y"])
@pytest.mark.parametrize("ny,nx", [(8, 32), (32, 32), (33, 31), (16, 12), (5, 100), (100, 5),
                                   (65, 64), (2, 3000), (71, 67)])
def test_grid_shapes(q, ctx, precision, order, ny, nx):
    px, py = grid(ny, nx, order)
    run(q, ctx, px, py, 37, 3, 1, precision, name=f"grid {ny}x{nx} {order}")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("K,R,R_block,mode", [(1, 2, 1, 0), (8, 5, 1, 1), (130, 600, 1, 0),
                                              (513, 9, 2, 0), (66, 7, 4, 1), (129, 5, 3, 0)])
def test_grid_frequencies(q, ctx, precision, K, R, R_block, mode):
    px, py = grid(32, 32, "x", 1)
    run(q, ctx, px, py, K, R, R_block, precision, mode, name="frequencies")


@pytest.mark.parametrize("R", [2, 520])
def test_large_tiles(q, ctx, R):
    px, py = grid(66, 70, "y", 2)
    run(q, ctx, px, py, 21, R, 1, 0, name="large tiles")


def test_given_coefficients(q, ctx):
    px, py = grid(20, 30, "x", 3)
    coef = np.random.default_rng(1).normal(size=(6, 2 * 77))
    run(q, ctx, px, py, 77, 6, 1, 0, coef=coef, name="given")


def not_quite(kind):
    px, py = grid(40, 48, "x", 4)
    if kind == "moved":  # one point off by one unit in the last place, late in the list
        px[-3] = np.nextafter(px[-3], 9.0)
    elif kind == "short":
        px, py = px[:-1], py[:-1]
    elif kind == "line":
        py[:] = 0.25
    elif kind == "same":
        px[:], py[:] = 1.5, 0.25
    elif kind == "disk":
        keep = px * px + py * py < 6.0
        px, py = px[keep], py[keep]
    elif kind == "ragged":  # rows of the same length, but shifted
        px = px + 0.01 * py
    elif kind == "first":
        py[0] += 1.0
    elif kind == "random":
        px = np.random.default_rng(0).uniform(-3, 3, px.size)
    return px, py


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["moved", "short", "line", "same", "disk", "ragged", "first",
                                  "random"])
def test_points_that_are_no_grid(q, ctx, precision, kind):
    px, py = not_quite(kind)
    run(q, ctx, px, py, 45, 4, 1, precision, name=kind)


def test_points_change_between_replays(q, ctx):
    """Captured once; the points' values change in place between replays
    from a grid to none and back."""
    K, R, P = 50, 4, 1024
    a, b = grid(32, 32, "x", 5), (np.random.default_rng(2).uniform(-3, 3, P),) * 2
    s = q.logpolar_sampler(1e-3, 1e2)
    fx, fy, area = ctx.sample_frequencies(s, R, K)
    w = ctx.weights(q.psd(0.1, 25.0), fx, fy, area)
    px, py = dev(a[0]), dev(a[1])
    out = torch.empty((R, P), dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.synthesize_phase(K, fx, fy, w, px, py, R, 1, rng=q.Rng(1, 0, 0), precision=0, out=out)
    for pts in (a, b, a, b):
        px.copy_(dev(pts[0]))
        py.copy_(dev(pts[1]))
        out.fill_(float("nan"))
        g.replay()
        ref = oracle.synthesize(host(fx), host(fy), host(w), pts[0], pts[1], R, 1, K=K, seed=1)
        assert np.max(np.abs(host(out) - ref)) <= 1e-11 * math.sqrt(np.mean(ref * ref))
