"""The backward pass of the scan where it is walked chunk by chunk (d and m up to 128): sizes around the tiles of sixteen, one to a few
chunks, states narrower and wider than the factors, rows in units of their own; against the oracle's adjoint recurrence."""
import math

import numpy as np
import pytest

from test_gpu_parity import G, dev, host, say  # noqa: F401

pytestmark = pytest.mark.gpu


def run(G, oracle, T, d, m, batch, chunk, ctype, with_init, units=None):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(1000 * d + m + T)
    # near the identity, so that the adjoints' sums cancel little
    Z = oracle.to_goom((np.eye(d) + 0.5 / np.sqrt(d) * rng.standard_normal((batch, T, d, d))).astype(comp))
    S0 = oracle.to_goom(rng.standard_normal((batch, d, m)).astype(comp)) if with_init else None
    Gp = rng.standard_normal((batch, T, d, m)).astype(comp)
    if d > 1:
        Z[:, T // 2, 0, d - 1] = -np.inf  # a zero entry
        Gp[:, T // 3, d - 1, 0] = 0.0     # an entry the loss does not see
    if units is not None:  # row i of every state in units of e^units[i]: the gradients stay what they are
        Z = (Z + (units[:, None] - units[None, :])).astype(ctype)
        S0 = (S0 + units[:, None]).astype(ctype)
    say(f"scan adjoint T={T} d={d} m={m} batch={batch} chunk={chunk} {np.dtype(ctype).name}")
    Pd = G.scan(dev(Z), None if S0 is None else dev(S0))
    P = host(Pd)
    gm, gi = G.scan_backward(dev(Z), Pd, dev(Gp), None if S0 is None else dev(S0), chunk_len=chunk)
    gm = host(gm).astype(np.float64)
    # Each of the T sums of d + m products that an adjoint passes through is rounded: sqrt(T (d + m)) roundings of 2^-24 (2^-53) of the
    # terms, which on these inputs are at most some 50 times their sum; a float log-magnitude of size s is itself good to s 2^-24.
    eta = 2.0 ** -24 if comp == np.float32 else 2.0 ** -53
    size = 1.0 if units is None else 2.0 * np.abs(units).max()
    bound = 50 * eta * (math.sqrt(T * (d + m)) + size) + 8 * eta
    for b in range(batch):
        wm, wi, _ = oracle.scan_backward(Z[b], Gp[b], init=None if S0 is None else S0[b], p=P[b])
        err = np.abs(gm[b] - wm).max(axis=(1, 2)) / np.abs(wm).max()
        assert err.max() <= bound, (b, int(err.argmax()), err.max(), bound)
        if with_init:
            e0 = np.abs(host(gi)[b].astype(np.float64) - wi).max() / np.abs(wi).max()
            assert e0 <= bound, (b, e0, bound)
        if d > 1:
            assert np.all(gm[b, T // 2, 0, d - 1] == 0.0)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [1, 2, 15, 16, 17, 31, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 127, 128])
def test_sizes(G, oracle, d, ctype):  # noqa: F811
    run(G, oracle, 19, d, d, 2, 8, ctype, d % 2 == 0)  # three chunks, the last one shorter
    run(G, oracle, 8, d, d, 1, 8, ctype, d % 2 == 1)   # one chunk


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d,m", [(20, 1), (64, 3), (33, 16), (16, 33), (5, 100), (100, 17), (128, 1), (1, 128)])
def test_states_of_another_width(G, oracle, d, m, ctype):  # noqa: F811
    run(G, oracle, 21, d, m, 2, 5, ctype, True)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("T,chunk", [(1, 0), (2, 1), (9, 8), (64, 0), (65, 1)])
def test_lengths(G, oracle, T, chunk, ctype):  # noqa: F811
    run(G, oracle, T, 24, 24, 3, chunk, ctype, False)


# rows e^40 (in double e^400) apart: the adjoints' rows lie as far apart the other way, the sums over a state's columns have to keep them
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [12, 40, 64, 100])
def test_rows_in_units_of_their_own(G, oracle, d, ctype):  # noqa: F811
    units = np.rint(np.linspace(-1.0, 1.0, d) * (20.0 if ctype == np.complex64 else 200.0))
    run(G, oracle, 20, d, d, 1, 8, ctype, True, units)
    run(G, oracle, 20, d, d, 1, 0, ctype, True, np.random.default_rng(d).permutation(units))


# matrices that are mostly padding, in many chunks: the workspace that the query names holds them all
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [1, 2])
def test_tiny_matrices_in_many_chunks(G, oracle, d, ctype):  # noqa: F811
    G.profile_enable(True)
    run(G, oracle, 1500, d, d, 1, 0, ctype, True)
    assert "scan_adjoint_carries" in [label for label, _ in G.profile_records()]
    G.profile_enable(False)
