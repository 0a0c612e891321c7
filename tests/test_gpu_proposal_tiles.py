"""The proposal's kernels at the edges of their row tiles (48 rows in training,
64 forward, one block per compute unit) against the FP64 oracle: single rows,
one row more or less than a tile, blocks of several tiles whose last is ragged,
grids longer than a tile, more contexts than lanes.

Tolerances as for the whole path: 1e-5 of the output scale (forward), 1e-5
(loss), 1e-5 normwise (gradient).
"""
import math

import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu

LMIN, LW = math.log(workloads.FMIN), math.log(workloads.FMAX / workloads.FMIN)


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


def params(seed):
    rng = np.random.default_rng(seed)
    prm = workloads.mlp_init(seed, scale=1.0) * 0.3
    return (prm + rng.normal(0, 0.02, prm.size)).astype(np.float32)


@pytest.mark.parametrize("n_ctx,m,G", [(1, 1, 1), (1, 47, 1), (2, 24, 65), (3, 17, 33), (70, 5, 100),
                                       (7, 2048, 64), (9, 3001, 129), (16, 2100, 32)])
def test_step_tiles(q, ctx, n_ctx, m, G):
    prm = params(n_ctx + m)
    c4 = workloads.proposal_contexts(n_ctx, seed=m)
    ell, theta, h = oracle.proposal_rows(c4, m, 0.1, workloads.FMIN, workloads.FMAX, index=3)
    p = q.Proposal(ctx, workloads.FMIN, workloads.FMAX, prm)
    print(f"step n_ctx{n_ctx} m{m} G{G}", flush=True)
    loss, grad = p.loss_grad(dev(c4), dev(ell), dev(theta), dev(h), G=G)
    rl, rg = oracle.mlp_loss_grad(prm.astype(np.float64), c4, ell, theta, h, LMIN, LW, G=G)
    torch.cuda.synchronize()
    e = np.linalg.norm(grad.double().cpu().numpy() - rg) / np.linalg.norm(rg)
    print(f"  loss {loss:.8f} vs {rl:.8f}; gradient {e:.2e}", flush=True)
    assert loss == pytest.approx(rl, rel=1e-5, abs=1e-6)
    assert e < 1e-5
    p.close()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 40000])
def test_forward_tiles(q, ctx, n):
    prm = params(n)
    rng = np.random.default_rng(n)
    p = q.Proposal(ctx, workloads.FMIN, workloads.FMAX, prm)
    ell = rng.uniform(LMIN, LMIN + LW, n)
    c4 = np.stack([rng.uniform(0.5, 10, n), rng.uniform(10, 100, n), rng.uniform(1, 130, n),
                   rng.uniform(0, np.pi, n)], 1)
    print(f"forward n{n}", flush=True)
    out = p.forward(dev(ell), dev(c4))
    torch.cuda.synchronize()
    ref = oracle.mlp_forward(prm.astype(np.float64), ell, c4, LMIN, LW)
    assert np.max(np.abs(out.double().cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
    p.close()
