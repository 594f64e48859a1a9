"""Scaled exponentiation of float vectors, four entries a lane (16 to 64 entries, multiples of four, 16-byte aligned) and one a lane: sizes at the
edges of the two, one vector and a number that no workgroup divides, zeros, infinities, NaN, and operands that begin between 16-byte steps."""
import numpy as np
import pytest
import torch

from test_gpu_parity import G, dev, host  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [12, 15, 16, 20, 31, 32, 36, 60, 64, 65, 68])
@pytest.mark.parametrize("n", [1, 7, 1001])
def test_sizes_and_alignment(G, oracle, d, n):  # noqa: F811
    rng = np.random.default_rng(1300 + d + n)
    z = (rng.normal(0.0, 300.0, (n, d)) + 1j * np.pi * rng.integers(0, 2, (n, d))).astype(np.complex64)
    z.real[rng.random((n, d)) < 0.1] = -np.inf
    z.real[n // 2, :] = -np.inf  # a vector of zeros
    want, cw = oracle.scaled_exp(z)
    eps = np.finfo(np.float32).eps
    odd = torch.empty(n * d + 1, dtype=torch.complex64, device="cuda")[1:].view(n, d)  # 8 bytes from a 16-byte step
    odd.copy_(dev(z))
    for zd in (dev(z), odd):
        got, c = (host(v) for v in G.scaled_exp(zd, want_logscale=True))
        assert np.array_equal(c, cw.astype(np.float32))
        assert np.all(np.abs(got - want) <= 4 * eps * np.abs(want) + np.finfo(np.float32).tiny)
        assert np.array_equal(got, host(G.scaled_exp(zd)))


@pytest.mark.parametrize("d", [16, 32, 64])
def test_not_finite(G, d):  # noqa: F811
    """A NaN is passed by and comes out as zero, as the log scale where it is the first entry; beside +inf all other entries vanish."""
    z = np.zeros((4, d), dtype=np.complex64)
    z.real[0, 3] = z.real[1, 0] = np.nan
    z.real[2, 5] = np.inf
    got, c = (host(v) for v in G.scaled_exp(dev(z), want_logscale=True))
    e2 = np.float32(np.exp(2.0))
    ones = np.full(d, e2)
    first = ones.copy()
    first[3] = 0
    assert np.array_equal(got[0], first) and c[0] == 0
    assert got[1, 0] == 0 and np.array_equal(got[1, 1:], ones[1:]) and np.isnan(c[1])
    assert np.isnan(got[2, 5]) and np.all(np.delete(got[2], 5) == 0) and c[2] == np.inf
    assert np.array_equal(got[3], ones) and c[3] == 0
