"""The memory of calls that fill the device only with the help of frequency
ranges or of the two-phase kernel's tiles: eager calls must leave the workspace
that a captured graph holds alone, must not wait for the device, and must do
without where no memory is to be had.  Fields against the FP64 oracle or, bit for
bit, against the same call alone; tolerances as for the whole contraction.
"""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TOL = {0: 1e-11, 1: 1e-5, 4: 1e-5}


@pytest.fixture(scope="module")
def q():
    import paper_2404_02978_amd as q
    q.load_library()
    return q


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.double().cpu().numpy()


def problem(ctx, q, K, R, R_block, P, seed=1):
    rng = np.random.default_rng([K, P, seed])
    s = q.logpolar_sampler(1e-3, 1e2, index=3)
    fx, fy, area = ctx.sample_frequencies(s, math.ceil(R / R_block), K)
    w = ctx.weights(q.psd(0.1, 25.0), fx, fy, area)
    return fx, fy, w, dev(rng.uniform(-4, 4, P)), dev(rng.uniform(-4, 4, P))


def output(R, P, precision):
    return torch.zeros((R, P), dtype=torch.float64 if precision == 0 else torch.float32,
                       device="cuda")


@pytest.mark.parametrize("K,R,R_block,P", [(4096, 128, 128, 1024), (10007, 259, 259, 3000)])
def test_eager_calls_leave_a_captured_workspace_alone(q, K, R, R_block, P):
    """A captured screen that fills the device holds the workspace; eager calls
    that want ranges (first case) or two-phase tiles (second) run between its
    replays, and so do allocations that would take the memory if it were freed."""
    big = (1000, 256, 256, 131072)
    with q.Context(0) as c:
        fx, fy, w, px, py = problem(c, q, *big)
        out = output(big[1], big[3], 4)
        args = (big[0], fx, fy, w, px, py, big[1], big[2])
        kw = dict(rng=q.Rng(5, 0, 0), precision=4, out=out)
        c.synthesize_phase(*args, **kw)
        want = out.clone()
        torch.cuda.synchronize()
        print(f"capture {big}, eager K{K} R{R} P{P}", flush=True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            c.synthesize_phase(*args, **kw)
        small = problem(c, q, K, R, R_block, P, 2)
        ref = oracle.synthesize(*(host(v) for v in small[:3]), host(small[3])[:64],
                                host(small[4])[:64], R, R_block, K=K, seed=6)
        fill = []
        for _ in range(3):
            got = c.synthesize_phase(K, *small[:3], *small[3:], R, R_block, rng=q.Rng(6, 0, 0),
                                     precision=1)
            e = np.max(np.abs(host(got)[:, :64] - ref)) / math.sqrt(np.mean(ref * ref))
            assert e <= TOL[1]
            fill.append(torch.full((3 << 20,), 7.0, dtype=torch.float64, device="cuda"))
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            assert all(bool((f == 7.0).all()) for f in fill)


def test_scratch_grows_without_waiting(q):
    """A call that takes ranges for the first time returns while another stream
    is busy, and may be made while another stream is being captured."""
    K, R, P = 4096, 16, 512
    with q.Context(0) as c:
        fx, fy, w, px, py = problem(c, q, K, R, R, P)
        args = (K, fx, fy, w, px, py, R, R)
        busy, done, out = torch.cuda.Stream(), torch.cuda.Event(), output(R, P, 0)
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(200_000_000)  # a tenth of a second or more
            done.record()
        c.synthesize_phase(*args, rng=q.Rng(1, 0, 0), precision=0, out=out)
        assert not done.query()
        want = host(out)
    with q.Context(0) as c:
        other, x = torch.cuda.Stream(), torch.zeros(8, device="cuda")
        out.zero_()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            x += 1.0
            with torch.cuda.stream(other):
                c.synthesize_phase(*args, rng=q.Rng(1, 0, 0), precision=0, out=out)
            x += 1.0
        g.replay()
        assert np.array_equal(host(out), want) and float(x[0]) == 2.0


@pytest.mark.parametrize("precision", [0, 1, 4])
def test_capped_scratch_gives_way_to_the_workspace(q, precision):
    """Scratch first, then a workspace that needs the whole cap, then ranges
    without room."""
    K, R, R_block, P = 2100, 30, 30, 45
    with q.Context(0, workspace_cap=3 << 20) as c:
        fx, fy, w, px, py = problem(c, q, K, R, R_block, P)
        ref = oracle.synthesize(host(fx), host(fy), host(w), host(px), host(py), R, R_block, K=K,
                                seed=1)
        for n in (0, 90000, 0):
            if n:  # 4 doubles for every 256 points of a set: 2.9 MB
                s = q.logpolar_sampler(1e-3, 1e2)
                gx, gy, _ = c.sample_frequencies(s, n, 4)
                c.point_set_measures(gx, gy, n, 4, -100.0, -100.0, 200.0, 200.0, 0.1)
            out = c.synthesize_phase(K, fx, fy, w, px, py, R, R_block, rng=q.Rng(1, 0, 0),
                                     precision=precision)
            assert np.max(np.abs(host(out) - ref)) <= TOL[precision] * math.sqrt(np.mean(ref * ref))


def test_grid_answers_of_two_contexts(q):
    """512 calls in ranges on a grid's points, from each of two contexts on
    streams of their own that start together: every answer is its call's own, so
    every field is the same."""
    K, R, n, calls = 4096, 8, 32, 512
    with q.Context(0) as a, q.Context(0) as b:
        fx, fy, w, _, _ = problem(a, q, K, R, 1, 1)
        g = np.linspace(0.0, 1.0, n)
        px, py = dev(np.tile(g, n)), dev(np.repeat(g, n))
        outs = [torch.full((calls, R, n * n), float("nan"), dtype=torch.float64, device="cuda")
                for _ in range(2)]

        def call(c, out):
            c.synthesize_phase(K, fx, fy, w, px, py, R, 1, rng=q.Rng(2, 0, 0), precision=0, out=out)

        call(a, outs[0][0])
        call(b, outs[1][0])  # both hold their scratch now
        want = host(outs[0][0])
        start = torch.cuda.Event()
        torch.cuda._sleep(50_000_000)
        start.record()
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        for s in streams:
            s.wait_event(start)
        print("512 calls on each of two streams", flush=True)
        for c, s, o in zip((a, b), streams, outs):
            with torch.cuda.stream(s):
                for i in range(calls):
                    call(c, o[i])
        torch.cuda.synchronize()
        for o in outs:
            assert torch.equal(o, torch.as_tensor(want).cuda().expand_as(o))
        ref = oracle.synthesize(host(fx), host(fy), host(w), host(px), host(py), R, 1, K=K, seed=2)
        assert np.max(np.abs(want - ref)) <= TOL[0] * math.sqrt(np.mean(ref * ref))


def test_more_contexts_than_words_for_grids(q):
    """Contexts beyond the 512 words take the general kernel."""
    K, R, n = 1024, 8, 32
    held = [q.Context(0) for _ in range(514)]
    fx, fy, w, _, _ = problem(held[0], q, K, R, 1, 1)
    g = np.linspace(0.0, 1.0, n)
    px, py = dev(np.tile(g, n)), dev(np.repeat(g, n))
    ref = oracle.synthesize(host(fx), host(fy), host(w), host(px), host(py), R, 1, K=K, seed=2)
    for c in (held[0], held[-1]):
        out = c.synthesize_phase(K, fx, fy, w, px, py, R, 1, rng=q.Rng(2, 0, 0), precision=0)
        assert np.max(np.abs(host(out) - ref)) <= TOL[0] * math.sqrt(np.mean(ref * ref))
    for c in held:
        c.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_captured_grids_keep_their_route(q, precision):
    """A grid whose eager call would take ranges besides: the captured call goes
    through the rows and columns as well, which needs no memory, and gives the same
    bits; those of the general kernel differ (the points in another order)."""
    K, R, n = 4096, 64, 32
    with q.Context(0) as c:
        fx, fy, w, _, _ = problem(c, q, K, R, 1, 1)
        g = np.sort(np.random.default_rng(1).uniform(0.0, 1.0, n))
        x, y = np.tile(g, n), np.repeat(g, n)
        order = np.random.default_rng(0).permutation(n * n)
        px, py = dev(x), dev(y)
        outs = [output(R, n * n, precision) for _ in range(3)]
        kw = dict(rng=q.Rng(2, 0, 0), precision=precision)
        c.synthesize_phase(K, fx, fy, w, px, py, R, 1, out=outs[0], **kw)
        c.synthesize_phase(K, fx, fy, w, dev(x[order]), dev(y[order]), R, 1, out=outs[1], **kw)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            c.synthesize_phase(K, fx, fy, w, px, py, R, 1, out=outs[2], **kw)
        print(f"grid p{precision}", flush=True)
        for _ in range(2):
            outs[2].fill_(float("nan"))
            graph.replay()
            assert np.array_equal(host(outs[2]), host(outs[0]))
        general = np.empty_like(host(outs[1]))
        general[:, order] = host(outs[1])
        assert not np.array_equal(general, host(outs[0]))


def test_full_problem_without_room_for_ranges(q):
    """A screen that fills the device, whose 513 tiles would run better in two
    ranges, in a context with room for its tiles but not for 136 MB of partial
    sums besides: one range."""
    K, R, P = 4096, 130, 131100
    with q.Context(0, workspace_cap=160 << 20) as c:
        fx, fy, w, px, py = problem(c, q, K, R, R, P)
        s = q.logpolar_sampler(1e-3, 1e2)
        n = 1100000  # a workspace of 35.2 MB
        gx, gy, _ = c.sample_frequencies(s, n, 4)
        c.point_set_measures(gx, gy, n, 4, -100.0, -100.0, 200.0, 200.0, 0.1)
        print(f"full K{K} R{R} P{P}", flush=True)
        out = c.synthesize_phase(K, fx, fy, w, px, py, R, R, rng=q.Rng(1, 0, 0), precision=1)
        sel = np.r_[0:8, P - 8:P]
        ref = oracle.synthesize(host(fx), host(fy), host(w), host(px)[sel], host(py)[sel], R, R,
                                K=K, seed=1)
        assert np.max(np.abs(host(out)[:, sel] - ref)) <= TOL[1] * math.sqrt(np.mean(ref * ref))


@pytest.mark.parametrize("precision", [0, 1])
def test_captured_time_series_in_the_smaller_workspace(q, precision):
    """A workspace with room for the estimator's longer blocks only, which cannot
    grow under capture."""
    K, M, R, R_block = 64, 1024, 2000, 50
    with q.Context(0) as c:
        args = (q.psd(0.1, 25.0), q.Aperture(8.0, 1.1), (0.0, 0.0), (56.5, 0.0), (10.2, 0.0), 1e-3, M)
        tail = (K, R, R_block)
        kw = dict(rng=q.Rng(3, 0, 0), precision=precision)
        # 4.1 MB of partial sums (8.2 in shorter blocks) and 16.4 MB of pistons, of
        # two telescopes in FP32, of their differences in FP64; frequencies
        n = 670000  # 21.4 MB
        gx, gy, _ = c.sample_frequencies(q.logpolar_sampler(1e-3, 1e2), n, 4)
        c.point_set_measures(gx, gy, n, 4, -100.0, -100.0, 200.0, 200.0, 0.1)
        torch.cuda.synchronize()
        print(f"series p{precision}", flush=True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            sf, se = c.temporal_piston_structure(*args, q.cartesian_sampler(8, 0.25 / 22.0), *tail,
                                                 **kw)
        for _ in range(2):
            sf.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            with q.Context(0) as other:
                ref, ref_se = other.temporal_piston_structure(
                    *args, q.cartesian_sampler(8, 0.25 / 22.0), *tail, **kw)
            assert np.allclose(host(sf), host(ref), rtol=1e-12, atol=0)
            assert np.allclose(host(se), host(ref_se), rtol=1e-9, atol=0)
