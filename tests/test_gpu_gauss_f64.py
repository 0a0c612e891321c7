"""Accuracy of the binary64 Gaussian coefficients, read back bit for bit: with one
frequency (1, 0) of weight 1, the field is a at the origin and b at (1/4, 0).  Of
a million pairs, from the narrow kernels' generator (one realisation per set) and
from the tabulated one of shared sets, against extended precision (64 bits of
mantissa) on the same Philox words.

Bounds, in units of the pair's radius: what sqrt(-2 log u) and sincospi of the
device library give on the same million pairs, 3.04e-16 at most and 5.73e-17 RMS;
4.82e-16 and 6.57e-17 in the Eq. 3 mode, which multiplies two cosines.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

R = 1 << 20
LD = np.longdouble


@pytest.fixture(scope="module")
def q():
    import paper_2404_02978_amd as q
    q.load_library()
    return q


def philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 over arrays of first words (uint64 holding 32 bits)."""
    mask = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) + np.zeros_like(c1) for v in (c0, c1, c2, c3)]
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def exact(seed, mode):
    """a, b and their radius in extended precision."""
    real = np.arange(R, dtype=np.uint64)
    x = philox(0, real, 0, 0, seed, 0)
    u = [(LD(1) * (v >> np.uint64(9)).astype(LD) + LD(0.5)) / LD(1 << 23) for v in x[:3]]
    rho = np.sqrt(-2 * np.log(u[0]))
    turn = [2 * LD("3.14159265358979323846264338327950288") * (v - np.rint(v)) for v in u[1:]]
    if mode == 0:
        return rho * np.cos(turn[0]), rho * np.sin(turn[0]), rho
    g = np.sqrt(LD(2)) * rho * np.cos(turn[0])
    return g * np.cos(turn[1]), -g * np.sin(turn[1]), np.sqrt(LD(2)) * rho


def test_words_match_the_oracle():
    x = philox(0, np.arange(5, dtype=np.uint64), 0, 0, 17, 0)
    for r in range(5):
        want = oracle.philox4x32_10(np.array([0, r, 0, 0], dtype=np.uint32),
                                    np.array([17, 0], dtype=np.uint32))
        assert [int(v[r]) for v in x] == [int(v) for v in want]


@pytest.mark.parametrize("R_block", [1, R])
@pytest.mark.parametrize("mode", [0, 1])
def test_coefficients(q, R_block, mode):
    seed, n_sets = 17, R // R_block
    px = torch.tensor([0.0, 0.25], dtype=torch.float64, device="cuda")
    one = torch.ones(n_sets, dtype=torch.float64, device="cuda")
    zero = torch.zeros(max(n_sets, 2), dtype=torch.float64, device="cuda")
    print(f"R_block {R_block} mode {mode}", flush=True)
    with q.Context(0) as c:
        out = c.synthesize_phase(1, one, zero[:n_sets], one, px, zero[:2], R, R_block,
                                 rng=q.Rng(seed, 0, mode), precision=0)
        torch.cuda.synchronize()
    got = out.cpu().numpy()
    a, b, rho = exact(seed, mode)
    e = np.concatenate([(got[:, 0] - a) / rho, (got[:, 1] - b) / rho]).astype(float)
    rms = np.sqrt(np.mean(e * e))
    print(f"  max {np.abs(e).max():.3e} rms {rms:.3e}", flush=True)
    most, mean = ((3.04e-16, 5.73e-17), (4.82e-16, 6.57e-17))[mode]
    assert np.abs(e).max() <= most and rms <= mean
