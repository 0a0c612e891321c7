"""Accuracy of the proposal's kernels beyond the bounds of test_gpu_proposal.py:
the gradient with hundreds to thousands of rows per block, whose sums must not
lose what binary32 rounds away, against a binary64 reference in torch (checked
against the oracle here); and the hidden units' tanh.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu

LMIN, LW = math.log(workloads.FMIN), math.log(workloads.FMAX / workloads.FMIN)
HID = 128


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


def split(p):
    at = np.cumsum([0, 5 * HID, HID, HID * HID, HID, 2 * HID, 2])
    W1, b1, W2, b2, W3, b3 = (p[i:j] for i, j in zip(at, at[1:]))
    return W1.view(HID, 5), b1, W2.view(HID, HID), b2, W3.view(2, HID), b3


def reference(prm, c4, ell, theta, h, G):
    """Loss and gradient in binary64; the inputs are rounded to binary32, as the
    kernels' are."""
    p = prm.double().clone().requires_grad_(True)
    W1, b1, W2, b2, W3, b3 = split(p)

    def net(l, c):
        x = torch.stack([2 * (l - LMIN) / LW - 1, 2 * c[:, 3] / math.pi - 1, c[:, 0].log() / 4,
                         c[:, 1].log() / 4 - 1, c[:, 2].log() / 4 - 0.5], 1).float().double()
        return torch.tanh(torch.tanh(x @ W1.T + b1) @ W2.T + b2) @ W3.T + b3

    n, m = c4.shape[0], ell.numel() // c4.shape[0]
    at = torch.arange(n, device="cuda")
    H = h.sum()
    o = net(ell, c4[at.repeat_interleave(m)])
    C = torch.cos(2 * (theta - c4[:, 3].repeat_interleave(m)))
    loss = -(h / H * (o[:, 0] + torch.log1p(0.9 * torch.tanh(o[:, 1]) * C))).sum()
    g = (LMIN + (torch.arange(G, device="cuda", dtype=torch.float64) + 0.5) * LW / G).repeat(n)
    og = net(g, c4[at.repeat_interleave(G)])[:, 0].view(n, G)
    logZ = torch.logsumexp(og, 1) + math.log(LW / G)
    loss = loss + (h.view(n, m).sum(1) / H * logZ).sum()
    loss.backward()
    return loss.item(), p.grad


def step(q, ctx, n_ctx, m, G, seed):
    prm = workloads.mlp_init(seed, scale=1.0) * (1.0, 0.3)[seed % 2]
    prm = (prm + np.random.default_rng(seed).normal(0, 0.02, prm.size)).astype(np.float32)
    c4 = workloads.proposal_contexts(n_ctx, seed=seed)
    s = q.logpolar_sampler(workloads.FMIN, workloads.FMAX, index=1000 * seed)
    p = q.Proposal(ctx, workloads.FMIN, workloads.FMAX, prm)
    rows = p.rows(s, dev(c4), m, 0.1)
    loss, grad = p.loss_grad(dev(c4), *rows, G=G)
    ref = reference(torch.as_tensor(prm).cuda(), dev(c4), *rows, G)
    torch.cuda.synchronize()
    p.close()
    return prm, c4, rows, loss, grad, ref


def test_reference_matches_the_oracle(q, ctx):
    G = 33
    prm, c4, rows, _, _, (loss, grad) = step(q, ctx, 3, 200, G, 1)
    rl, rg = oracle.mlp_loss_grad(prm.astype(np.float64), c4, *(r.cpu().numpy() for r in rows),
                                  LMIN, LW, G=G)
    assert loss == pytest.approx(rl, rel=1e-9)
    assert np.linalg.norm(grad.cpu().numpy() - rg) <= 1e-6 * np.linalg.norm(rg)


# Each row's share is binary32 arithmetic (unit roundoff 6e-8), with errors of its
# own; their sum is exact but for the rows of a tile: five roundoffs normwise
@pytest.mark.parametrize("seed", [0, 1, 2, 3])
@pytest.mark.parametrize("n_ctx,m,G", [(16, 2048, 64), (16, 20000, 64), (64, 20000, 128)])
def test_gradient_of_many_rows(q, ctx, n_ctx, m, G, seed):
    print(f"step n_ctx{n_ctx} m{m} G{G} seed{seed}", flush=True)
    _, _, _, loss, grad, (rl, rg) = step(q, ctx, n_ctx, m, G, seed)
    e = ((grad.double() - rg).norm() / rg.norm()).item()
    print(f"  gradient {e:.2e}", flush=True)
    assert loss == pytest.approx(rl, rel=1e-8)
    assert e <= 3e-7


def test_tanh_of_the_hidden_units(q, ctx):
    """With no weights in the second layer the outputs are tanh of two of its
    biases, bit for bit.  Errors in [5/8, 1), where the exponential's and the
    quotient's show most, in units of the last place: the library's tanhf has 0.417
    RMS and at most 1.41 there; 8192 values give the RMS to 1 %."""
    x = np.linspace(0.625, 1.0, 8192, endpoint=False).astype(np.float32)
    prm = np.zeros(workloads.mlp_init(0).size, dtype=np.float32)
    W1, b1, W2, b2, W3, b3 = split(t := torch.as_tensor(prm).cuda())
    W3[0, 5] = W3[1, 77] = 1.0
    p = q.Proposal(ctx, workloads.FMIN, workloads.FMAX, prm)
    ell, c4 = dev([LMIN]), dev(workloads.proposal_contexts(1, seed=1))
    xs, out = torch.as_tensor(x).cuda(), []
    for i in range(0, x.size, 2):
        b2[5], b2[77] = xs[i], xs[i + 1]
        p.set_params(t)
        out.append(p.forward(ell, c4))
    got = torch.cat(out).flatten().double().cpu().numpy()
    p.close()
    ref = np.tanh(x.astype(np.float64))
    e = np.abs(got - ref) / np.spacing(ref.astype(np.float32)).astype(np.float64)
    print(f"rms {math.sqrt(np.mean(e * e)):.3f} max {e.max():.3f}", flush=True)
    assert math.sqrt(np.mean(e * e)) <= 0.435 and e.max() <= 1.42
