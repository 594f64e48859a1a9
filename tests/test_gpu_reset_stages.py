"""Reset scans whose boundaries are all reset: one wave per panel of sixteen columns, at the sizes around the panels, chains that end on
a boundary, just after one and before the first, against the recurrence in double; and columns that are nothing but rounding."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, dev, host, say  # noqa: F401

pytestmark = pytest.mark.gpu


def real(z):
    return np.exp(z.real.astype(np.float64)) * np.where(z.imag > 1.5, -1.0, 1.0)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
def test_every_boundary_reset(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(d)
    for T, every, batch, start in ((1, 8, 1, False), (5, 8, 2, True), (40, 8, 2, False), (45, 8, 1, True), (12, 1, 1, True)):
        J = (np.eye(d) + 0.3 / np.sqrt(d) * rng.standard_normal((batch, T, d, d))).astype(comp)
        S = (np.eye(d) + 0.3 / np.sqrt(d) * rng.standard_normal((batch, d, d))).astype(comp) if start else None
        if d > 2:
            J[:, T // 2, :, d // 2] *= 1e-3  # a column that shrinks at one step
        Jz, Sz = oracle.to_goom(J), oracle.to_goom(S) if start else None
        say(f"every boundary reset T={T} d={d} every={every} batch={batch} start={start} {np.dtype(ctype).name}")
        states, flags, growth = (host(v) for v in G.scan_reset(dev(Jz), dev(Sz) if start else None, chunk_len=every))
        alone = host(G.lyapunov_spectrum(dev(Jz), 1.0 / T, dev(Sz) if start else None, chunk_len=every))
        every = min(every, T)  # (a chunk is no longer than the chain)
        for q in range(batch):
            x, grown = (real(Sz[q]) if start else np.eye(d)), np.zeros(d)
            for t in range(T):
                x = real(Jz[q, t]) @ x
                if (t + 1) % every == 0:
                    x, r = np.linalg.qr(x)
                    grown += np.log(np.abs(np.diag(r)))
                    x *= np.sign(np.diag(r))
                assert flags[q, t] == ((t + 1) % every == 0)
                # (a state's float log-magnitudes are rounded once; a double factorisation is good to cond^2 2^-53 of a column, cond <= 1e4)
                assert np.abs(real(states[q, t]) - x).max() <= (2e-6 if comp == np.float32 else 1e-8) * np.abs(x).max(), (q, t)
            if T % every:
                grown += np.log(np.abs(np.diag(np.linalg.qr(x)[1])))
            assert np.abs(growth[q] - grown).max() <= 1e-7 * max(1.0, np.abs(grown).max())
        # the spectrum alone keeps no states at the boundaries: the same numbers
        assert np.allclose(alone, growth, rtol=1e-14, atol=0.0)


# diagonal chains whose columns differ by e^+-300, a zero column among them: exact in every column
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [5, 20, 40, 64])
def test_columns_far_apart_and_empty(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    T, every = 12, 4
    rng = np.random.default_rng(d)
    logs = np.linspace(-300.0, 300.0, d) / every + 0.1 * rng.standard_normal((T, d))
    z = np.full((1, T, d, d), -np.inf + 0j, dtype=ctype)
    k = np.arange(d)
    z[0, :, k, k] = logs.T.astype(comp)
    z[0, 3, d // 2, d // 2] = -np.inf
    growth = host(G.lyapunov_spectrum(dev(z), 1.0 / T, chunk_len=every))[0]
    want = z[0, :, k, k].real.astype(np.float64).sum(axis=1)
    keep = k != d // 2
    assert np.abs(growth[keep] - want[keep]).max() <= 1e-9 * np.abs(want[keep]).max()
    assert np.all(np.isfinite(growth))


# products of a few Gaussian matrices, seldom examined: a last column that is 1e-8 of its norm off the others, whose pivot, a difference of
# squares, comes out on either side of zero.  The column itself is still good to some digits, and so is its growth.
@pytest.mark.parametrize("T,d,every,thr,seed", [(90, 80, 3, 0.6, 62), (90, 80, 3, 0.6, 63), (90, 80, 3, 0.7, 62), (90, 80, 3, 0.7, 67), (90, 128, 2, 0.6, 65)])
def test_column_of_rounding_keeps_its_growth(G, oracle, T, d, every, thr, seed):  # noqa: F811
    from paper_2510_03426_amd import RESET_COLINEAR
    Jz = oracle.to_goom(si.normal_chain(si.BASE_SEED + seed, T, d))
    S0 = oracle.to_goom(si.normal_init(si.BASE_SEED + seed, d, d))
    _, flags, growth = (host(v) for v in G.scan_reset(dev(Jz), dev(S0), chunk_len=every, policy=RESET_COLINEAR, cos_threshold=thr))
    _, _, oflag, ogrowth = oracle.reset_scan(Jz, S0, check_every=every, policy=0, cos_threshold=thr)
    assert np.array_equal(flags, oflag)
    assert np.abs(growth - ogrowth).max() < 1e-3 * T


# One state, two kernels: a wave per panel where every boundary is reset, a wave with the whole state where a boundary is examined first.  With
# a threshold of zero the second resets every boundary too, and the two take the same operations in the same order: every bit is the same,
# also where some boundaries need a second factorisation (products of Gaussian matrices: some, nearly all and none of them).
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [2, 16, 17, 32, 33, 48, 64])
def test_same_bits_as_the_kernel_that_examines(G, oracle, d, ctype):  # noqa: F811
    from paper_2510_03426_amd import RESET_COLINEAR
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(d)
    for T, every, gain, start in ((60, 1, 1.0, False), (61, 2, 1.0, True), (62, 3, 1.0, True), (41, 4, 0.5, False), (40, 8, 0.2, True)):
        J = rng.standard_normal((2, T, d, d)) / np.sqrt(d)
        J = oracle.to_goom(((1.0 - gain) * np.eye(d) + gain * J).astype(comp))
        S = oracle.to_goom(rng.standard_normal((2, d, d)).astype(comp)) if start else None
        say(f"always against examined T={T} d={d} every={every} gain={gain} {np.dtype(ctype).name}")
        put = dev(S) if start else None
        a = [host(v) for v in G.scan_reset(dev(J), put, chunk_len=every)]
        b = [host(v) for v in G.scan_reset(dev(J), put, chunk_len=every, policy=RESET_COLINEAR, cos_threshold=0.0)]
        assert np.array_equal(a[1], b[1])
        assert np.array_equal(a[2], b[2]), np.abs(a[2] - b[2]).max()
        assert np.array_equal(a[0], b[0])
