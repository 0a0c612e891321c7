"""The kernel for fields on regular grids, at sizes whose calls do ask for it:
each of its tile shapes, both orders of the points, frequency ranges besides,
shared sets, the Eq. 3 mode, given coefficients, points that are no grid late in
the list, and points that change between replays of a graph.

A grid's fields differ in their last bits from the general kernel's, which takes
the same points in another order: so the tests see which one did the work.  Both
against the FP64 oracle at 48 of the points, within 1e-11 (FP64) and 1e-5 (FP32
class) of the RMS, as for the general kernels.
"""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TOL = {0: 1e-11, 1: 1e-5, 2: 1e-5, 3: 1e-5, 4: 1e-5}


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


def grid(ny, nx, order):
    rng = np.random.default_rng([ny, nx])
    x, y = np.sort(rng.uniform(-3, 3, nx)), np.sort(rng.uniform(-3, 3, ny))
    if order == "x":
        return np.tile(x, ny), np.repeat(y, nx)
    return np.repeat(x, ny), np.tile(y, nx)


def frequencies(q, ctx, K, R, R_block):
    s = q.logpolar_sampler(1e-3, 1e2, index=9)
    fx, fy, area = ctx.sample_frequencies(s, math.ceil(R / R_block), K)
    return fx, fy, ctx.weights(q.psd(0.1, 25.0), fx, fy, area)


def run(q, ctx, px, py, K, R, R_block, precision, on_grid, mode=0, given=False):
    fx, fy, w = frequencies(q, ctx, K, R, R_block)
    coef = np.random.default_rng(K).normal(size=(R, 2 * K)) if given else None
    kw = dict(coef=dev(coef)) if given else dict(rng=q.Rng(6, 21, mode))
    order = np.random.default_rng(P := px.size).permutation(P)
    print(f"P{P} K{K} R{R} Rb{R_block} p{precision} mode{mode} given{given}", flush=True)
    out = host(ctx.synthesize_phase(K, fx, fy, w, dev(px), dev(py), R, R_block,
                                    precision=precision, **kw))
    other = np.empty_like(out)
    other[:, order] = host(ctx.synthesize_phase(K, fx, fy, w, dev(px[order]), dev(py[order]), R,
                                                R_block, precision=precision, **kw))
    sel = np.unique(np.r_[0, P - 1, np.random.default_rng(1).integers(0, P, 46)])
    ref = oracle.synthesize(host(fx), host(fy), host(w), px[sel], py[sel], R, R_block, K=K, seed=6,
                            counter=21, mode=mode, coef=coef)
    for got in (out, other):
        e = np.max(np.abs(got[:, sel] - ref)) / math.sqrt(np.mean(ref * ref))
        print(f"  eps_max {e:.2e}", flush=True)
        assert e <= TOL[precision]
    assert np.array_equal(out, other) != on_grid


# tile shapes: 64 x 64; 32 x 32 in 4 waves; in 16 waves; 32 x 16 in 16 waves
# (the last with frequency ranges of the general kernel besides)
SHAPES = [((66, 70), 260), ((32, 32), 520), ((33, 31), 300), ((40, 25), 90)]


@pytest.mark.parametrize("order", ["x", "y"])
@pytest.mark.parametrize("precision", [0, 1, 4])
@pytest.mark.parametrize("shape,R", SHAPES)
def test_tiles(q, ctx, shape, R, precision, order):
    K = {260: 65, 520: 97, 300: 333, 90: 2050}[R] * (1 if precision == 0 else 4)
    run(q, ctx, *grid(*shape, order), K, R, 1, precision, True)


@pytest.mark.parametrize("K,R,R_block,shape,mode", [
    (4096, 8, 1, (32, 32), 0), (1031, 70, 2, (64, 48), 1), (2049, 30, 4, (64, 64), 0),
    (1500, 47, 3, (48, 64), 0), (1200, 40, 1, (5, 200), 1), (900, 60, 1, (300, 5), 0),
    (4001, 3, 1, (71, 67), 0)])
def test_sets_modes_and_ranges(q, ctx, K, R, R_block, shape, mode):
    run(q, ctx, *grid(*shape, "x"), K, R, R_block, 0, True, mode)


def test_given_coefficients(q, ctx):
    run(q, ctx, *grid(32, 32, "x"), 700, 120, 1, 0, True, given=True)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["moved", "last", "short", "wide", "disk", "sheared"])
@pytest.mark.parametrize("K,R", [(4096, 16), (1100, 200)])
def test_points_that_are_no_grid(q, ctx, K, R, kind, precision):
    """K = 4096: the general kernel works in frequency ranges."""
    px, py = grid(48, 64, "x")
    if kind == "moved":  # one point, between those that every block looks at
        px[2 * px.size // 3 + 1] = np.nextafter(px[2 * px.size // 3 + 1], 9.0)
    elif kind == "last":
        py[-1] = np.nextafter(py[-1], 9.0)
    elif kind == "short":
        px, py = px[:-1], py[:-1]
    elif kind == "wide":  # a grid, but rows of two points: too much padding
        px, py = grid(1500, 2, "x")
    elif kind == "disk":
        keep = px * px + py * py < 6.0
        px, py = px[keep], py[keep]
    else:
        px = px + 0.01 * py
    run(q, ctx, px, py, K, R, 1, precision, False)


def test_points_change_between_replays(q, ctx):
    K, R, P = 600, 200, 1024
    a, b = grid(32, 32, "x"), tuple(np.random.default_rng(2).uniform(-3, 3, (2, P)))
    fx, fy, w = frequencies(q, ctx, K, R, 1)
    px, py = dev(a[0]), dev(a[1])
    out = torch.empty((R, P), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.synthesize_phase(K, fx, fy, w, px, py, R, 1, rng=q.Rng(1, 0, 0), precision=0, out=out)
    sel = np.arange(0, P, 31)
    for pts in (a, a, b, a, b):
        px.copy_(dev(pts[0]))
        py.copy_(dev(pts[1]))
        out.fill_(float("nan"))
        g.replay()
        ref = oracle.synthesize(host(fx), host(fy), host(w), pts[0][sel], pts[1][sel], R, 1, K=K,
                                seed=1)
        got = host(out)
        assert np.max(np.abs(got[:, sel] - ref)) <= TOL[0] * math.sqrt(np.mean(ref * ref))
        assert np.all(np.isfinite(got))


def test_blocks_of_several_items(q, ctx):
    """Two tiles per realisation and half as many blocks: no block leaves its second
    tile because the first block has not answered yet (600 calls, whose fields all
    are the first one's)."""
    K, R = 333, 300
    px, py = grid(33, 31, "x")
    fx, fy, w = frequencies(q, ctx, K, R, 1)
    dx, dy = dev(px), dev(py)
    out = torch.empty((R, px.size), dtype=torch.float64, device="cuda")
    first, bad = None, torch.zeros((), dtype=torch.int64, device="cuda")
    for _ in range(600):
        out.fill_(float("nan"))
        ctx.synthesize_phase(K, fx, fy, w, dx, dy, R, 1, rng=q.Rng(6, 21, 0), precision=0, out=out)
        first = out.clone() if first is None else first
        bad += (out != first).sum()
    assert int(bad) == 0 and bool(torch.isfinite(first).all())


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["weight", "last weight", "coefficient", "nan"])
def test_values_that_are_not_finite(q, ctx, kind, precision):
    """Infinite and NaN weights and coefficients: the fields of the general kernel,
    infinite where the sum is."""
    K, R = (1100, 40) if precision == 0 else (8192, 40)
    px, py = grid(32, 32, "x")
    fx, fy, w = frequencies(q, ctx, K, R, 1)
    coef = np.random.default_rng(2).normal(size=(R, 2 * K))
    if kind == "weight":
        w[K // 3] = float("inf")
    elif kind == "last weight":
        w[R * K - 1] = -float("inf")
    elif kind == "coefficient":
        coef[1, K], coef[7, 2 * K - 1] = np.inf, -np.inf
    else:
        coef[R - 1, 64] = np.nan
    order = np.random.default_rng(0).permutation(px.size)
    print(f"{kind} p{precision}", flush=True)
    out = host(ctx.synthesize_phase(K, fx, fy, w, dev(px), dev(py), R, 1, coef=dev(coef),
                                    precision=precision))
    other = np.empty_like(out)
    other[:, order] = host(ctx.synthesize_phase(K, fx, fy, w, dev(px[order]), dev(py[order]), R, 1,
                                                coef=dev(coef), precision=precision))
    assert not np.isfinite(other).all()
    assert np.array_equal(out, other, equal_nan=True)
