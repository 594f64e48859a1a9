"""Spectra of chains with many chunks, walked in segments that are joined afterwards: sizes at the edges of the panels, a last chunk that is shorter, initial
states, several items, chunks that are factored twice, and chains whose segments do not join (walked in order then)."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, dev, host  # noqa: F401

pytestmark = pytest.mark.gpu


def chain(seed, T, d, dtype, spread=0.0):
    """Well separated directions that the matrices turn only slowly (spread: per step, between the first and the last)."""
    x = np.eye(d) + 0.15 / np.sqrt(d) * si.normal_f32(si.BASE_SEED + seed, 1, T * d * d).reshape(T, d, d)
    return (x * np.exp(np.linspace(spread, -spread, d))[:, None]).astype(dtype)


def in_order(G, z, s0=None, chunk_len=0):  # noqa: F811
    """The same growth from the scan that keeps every state."""
    return G.scan_reset(z, s0, chunk_len=chunk_len)[2]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("d,T,chunk,batch", [(1, 64, 1, 1), (3, 129, 2, 1), (15, 200, 2, 2), (16, 321, 5, 1), (17, 192, 3, 1), (31, 400, 4, 2), (32, 130, 2, 1), (32, 65, 1, 1),
                                             (20, 127, 1, 3)])
def test_spectrum(G, oracle, d, T, chunk, batch, dtype):  # noqa: F811
    x = np.stack([chain(2000 + d + i, T, d, dtype, 0.05) for i in range(batch)])
    z = oracle.to_goom(x)
    lam = host(G.lyapunov_spectrum(dev(z), 0.01, chunk_len=chunk))
    kept = host(in_order(G, dev(z), chunk_len=chunk)) / (0.01 * T)
    for i in range(batch):
        ref = oracle.lyapunov_qr(np.exp(z[i].real.astype(np.float64)) * np.where(z[i].imag > 1.5, -1.0, 1.0), 0.01)
        # both sum T logarithms of numbers good to a few units of 2^-52, magnified by what the joining lost (1e6 at most)
        assert np.abs(lam[i] - ref).max() <= 1e-9 * max(1.0, np.abs(ref).max())
        assert np.abs(lam[i] - kept[i]).max() <= 1e-9 * max(1.0, np.abs(ref).max())


# from the first number of chunks on that is walked in segments, and one more
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("d,T,chunk,batch", [(1, 80, 1, 1), (3, 181, 2, 1), (16, 401, 5, 1), (17, 240, 3, 1), (32, 170, 2, 1), (32, 81, 1, 1)])
def test_spectrum_of_few_segments(G, oracle, d, T, chunk, batch, dtype):  # noqa: F811
    test_spectrum(G, oracle, d, T, chunk, batch, dtype)


def growth_in_extended_precision(x):
    """Logarithms of the triangular factors' diagonals, step by step."""
    Q, out = np.eye(x.shape[-1], dtype=np.longdouble), 0
    for M in x:
        Z = M @ Q
        norm = np.empty(len(Q), dtype=np.longdouble)
        for k in range(len(Q)):
            for _ in range(2):
                Z[:, k] -= Z[:, :k] @ (Z[:, :k].T @ Z[:, k])
            norm[k] = np.sqrt((Z[:, k] ** 2).sum())
            Z[:, k] /= norm[k]
        Q, out = Z, out + np.log(norm)
    return out.astype(np.float64)


@pytest.mark.parametrize("dtype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [8, 24, 32])
def test_weakly_separated_directions(G, d, dtype):  # noqa: F811
    """Segments that begin far from the chain's states, and joins that would magnify their roundings: as good as in order."""
    C, L = 96, 8
    for seed in range(3):
        x = np.eye(d) + 0.15 / np.sqrt(d) * np.random.default_rng(seed + d).standard_normal((C * L, d, d))
        z = (np.log(np.abs(x)) + 1j * np.pi * (x < 0)).astype(dtype)
        want = growth_in_extended_precision(np.exp(z.real.astype(np.longdouble)) * np.where(z.imag > 1, -1, 1))
        got = host(G.lyapunov_spectrum(dev(z[None]), 1.0 / (C * L), chunk_len=L))[0]
        # a chunk's factorisation: some units of 2^-52, times the spread of its columns (up to five); they add up as their number, at worst
        assert np.abs(got - want).max() <= 5 * 2.0 ** -52 * C, (seed, np.abs(got - want).max())


@pytest.mark.parametrize("d", [9, 32])
def test_initial_state_and_chunks_factored_twice(G, oracle, d):  # noqa: F811
    T, chunk = 640, 8
    z = dev(oracle.to_goom(chain(2100 + d, T, d, np.float32, 1.2)[None]))  # a chunk's columns lie e^-19 apart
    s0 = dev(oracle.to_goom(si.normal_f32(si.BASE_SEED + 2200 + d, 2, d * d).reshape(1, d, d)))
    lam = host(G.lyapunov_spectrum(z, 0.01, s0=s0, chunk_len=chunk))
    kept = host(in_order(G, z, s0, chunk_len=chunk)) / (0.01 * T)
    assert np.abs(lam - kept).max() <= 1e-8 * np.abs(kept).max()


# every direction grows alike, so that no segment's state comes close to the chain's (in order after all: the same bits); a chunk that loses a direction,
# whose growth is rounding from there on, and one that loses them all
@pytest.mark.parametrize("kind", ["turns", "singular", "zero"])
@pytest.mark.parametrize("d", [8, 24])
def test_segments_that_do_not_join(G, oracle, d, kind):  # noqa: F811
    T, chunk = 256, 3
    if kind == "turns":
        x = np.roll(np.eye(d), 1, axis=0)[None].repeat(T, 0) * np.float64(1.25)
    else:
        x = chain(2300 + d, T, d, np.float64)
        x[100, :, 2 if kind == "singular" else slice(None)] = 0.0
    z = dev(oracle.to_goom(x.astype(np.float32)[None]))
    lam = host(G.lyapunov_spectrum(z, 0.01, chunk_len=chunk))
    kept = host(in_order(G, z, chunk_len=chunk)) * (1.0 / (0.01 * T))
    if kind == "singular":
        assert np.abs(lam[:, :-1] - kept[:, :-1]).max() < 1e-9 and lam[0, -1] < -10.0 and kept[0, -1] < -10.0
    else:
        assert np.allclose(lam, kept, rtol=1e-14, atol=0.0, equal_nan=True)
