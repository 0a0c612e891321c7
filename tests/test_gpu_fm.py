"""The binary64 contraction of shared sets at the edges of its tiles: rows on
either side of 16 and 32 per wave and of the row waves' share, columns on either
side of 16, 32 and 64, ragged chunks of frequencies, both coefficient modes and
given coefficients, stored and squared, against the FP64 oracle.

Tolerance as for the whole FP64 path: 1e-11 of the RMS of the oracle's field,
and through the square 1e-10 of a structure function.
"""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


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


def problem(q, ctx, K, R, R_block, P):
    rng = np.random.default_rng([K, R, P])
    s = q.logpolar_sampler(1e-3, 1e2, index=5)
    fx, fy, area = ctx.sample_frequencies(s, math.ceil(R / R_block), K)
    w = ctx.weights(q.psd(0.1, 25.0), fx, fy, area)
    return fx, fy, w, rng.uniform(-3, 3, P), rng.uniform(-3, 3, P)


@pytest.mark.parametrize("mode", [0, 1, "given"])
@pytest.mark.parametrize("K,R,R_block,P", [(1, 9, 9, 1), (9, 16, 16, 16), (63, 34, 17, 17),
                                           (64, 64, 32, 32), (65, 99, 33, 33), (200, 65, 65, 64),
                                           (131, 300, 129, 65), (77, 2000, 2000, 31),
                                           (40, 9000, 9000, 130)])
def test_fields(q, ctx, K, R, R_block, P, mode):
    fx, fy, w, px, py = problem(q, ctx, K, R, R_block, P)
    coef = np.random.default_rng(K).normal(size=(R, 2 * K)) if mode == "given" else None
    kw = dict(coef=dev(coef)) if mode == "given" else dict(rng=q.Rng(11, 1 << 33, mode))
    print(f"field K{K} R{R} Rb{R_block} P{P} {mode}", flush=True)
    out = ctx.synthesize_phase(K, fx, fy, w, dev(px), dev(py), R, R_block, precision=0, **kw)
    ref = oracle.synthesize(host(fx), host(fy), host(w), px, py, R, R_block, K=K, seed=11,
                            counter=1 << 33, mode=0 if mode == "given" else mode, coef=coef)
    assert np.max(np.abs(host(out) - ref)) <= 1e-11 * math.sqrt(np.mean(ref * ref))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("K,R,R_block,P", [(65, 34, 17, 3), (130, 99, 33, 33), (77, 1000, 1000, 32),
                                           (40, 70000, 35000, 65)])
def test_structure_functions(q, ctx, K, R, R_block, P, mode):
    """The last has more than 1024 tiles of rows, which are added in two passes."""
    fx, fy, w, px, py = problem(q, ctx, K, R, R_block, P)
    print(f"sf K{K} R{R} Rb{R_block} P{P} {mode}", flush=True)
    sf, err = ctx.diff_piston_structure_sets(K, fx, fy, w, dev(px), dev(py), R, R_block,
                                             rng=q.Rng(3, 8, mode), precision=0)
    at = [oracle.synthesize(host(fx), host(fy), host(w), x, y, R, R_block, K=K, seed=3, counter=8,
                            mode=mode) for x, y in ((px, py), (np.zeros(1), np.zeros(1)))]
    d2 = (at[0] - at[1]) ** 2
    ref = d2.mean(0)
    assert np.max(np.abs(host(sf) - ref)) <= 1e-10 * np.max(ref)
    assert np.max(np.abs(host(err) - d2.std(0, ddof=1) / math.sqrt(R))) <= 1e-10 * np.max(ref)
