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


# Magnitudes further apart than a mantissa reaches: what the walk cannot hold is written again with an exponent an entry.
def reals(ctype):
    return np.float32 if ctype == np.complex64 else np.float64


def states(oracle, Z, S0):
    re, sg = oracle.scan(Z, S0)
    return (re + 1j * np.pi * sg).astype(Z.dtype)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_one_step_of_rows_far_apart(G, oracle, ctype):  # noqa: F811
    say(f"scan adjoint, one diagonal step, {np.dtype(ctype).name}")
    far = 60.0 if ctype == np.complex64 else 500.0
    Z = np.full((1, 1, 2, 2), -np.inf, dtype=ctype)
    Z[0, 0, 0, 0], Z[0, 0, 1, 1] = far, -far
    S0 = np.zeros((1, 2, 1), dtype=ctype)
    gm, gi = G.scan_backward(dev(Z), G.scan(dev(Z), dev(S0)), dev(np.ones((1, 1, 2, 1), dtype=reals(ctype))), dev(S0))
    # one term an entry, with one rounding of each of its three factors' exponentials
    assert np.allclose(host(gm)[0, 0], np.eye(2), rtol=0, atol=16 * np.finfo(reals(ctype)).eps)
    assert np.allclose(host(gi)[0, :, 0], 1.0, rtol=0, atol=16 * np.finfo(reals(ctype)).eps)


# rows e^120 (in double e^1000) apart, every row of every gradient against its own terms; of three chains one, so that the others keep the walk's
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d,m,chunk", [(3, 2, 0), (12, 12, 8), (33, 20, 8), (64, 64, 0), (100, 17, 7), (128, 128, 8)])
def test_rows_beyond_a_mantissa(G, oracle, d, m, chunk, ctype):  # noqa: F811
    say(f"scan adjoint, rows far apart, d={d} m={m} {np.dtype(ctype).name}")
    comp, T, batch, far = reals(ctype), 20, 3, 60.0 if ctype == np.complex64 else 500.0
    rng = np.random.default_rng(17 * d + m)
    Z = oracle.to_goom((np.eye(d) + 0.5 / np.sqrt(d) * rng.standard_normal((batch, T, d, d))).astype(comp))
    S0 = oracle.to_goom(rng.standard_normal((batch, d, m)).astype(comp))
    Gp = rng.standard_normal((batch, T, d, m)).astype(comp)
    units = rng.permutation(np.rint(np.linspace(-far, far, d)))
    Z[1] = (Z[1] + (units[:, None] - units[None, :])).astype(ctype)
    S0[1] = (S0[1] + units[:, None]).astype(ctype)
    P = np.stack([states(oracle, Z[b], S0[b]) for b in range(batch)])
    gm, gi = G.scan_backward(dev(Z), dev(P), dev(Gp), dev(S0), chunk_len=chunk)
    gm, gi = host(gm).astype(np.float64), host(gi).astype(np.float64)
    eta = np.finfo(comp).eps / 2
    # as in run() above, of the terms: |M_ij| sum_k |Lam_ik| |P_jk|, the largest of a row (log-magnitudes of up to 2 far are good to that times eta)
    bound = 50 * eta * (math.sqrt(T * (d + m)) + 4 * far)
    for b in range(batch):
        wm, wi, (lre, _) = oracle.scan_backward(Z[b], Gp[b], init=S0[b], p=P[b])
        prev = np.concatenate([S0[b][None], P[b][:-1]]).real
        for t in range(T):
            a = lre[t].reshape(d, m)[:, None, :] + prev[t][None, :, :]
            terms = np.exp(Z[b, t].real[..., None] + a).sum(-1).max(1)
            err = np.abs(gm[b, t] - wm[t]).max(1) / terms
            assert err.max() <= bound, (b, t, int(err.argmax()), err.max(), bound)
        e0 = np.abs(gi[b] - wi).max() / np.abs(wi).max()
        assert e0 <= bound, (b, e0, bound)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_diagonal_chain_in_chunks(G, oracle, ctype):  # noqa: F811
    say(f"scan adjoint, diagonal chain, {np.dtype(ctype).name}")
    T, d, m = 40, 5, 3
    Z = np.full((1, T, d, d), -np.inf, dtype=ctype)
    for i, s in enumerate((30.0, 0.0, -30.0, 7.0, -200.0)):
        Z[0, :, i, i] = s
    S0 = np.zeros((1, d, m), dtype=ctype)
    Gp = np.random.default_rng(3).integers(-8, 9, (1, T, d, m)).astype(reals(ctype))
    gm, gi = G.scan_backward(dev(Z), dev(states(oracle, Z[0], S0[0])[None]), dev(Gp), dev(S0), chunk_len=8)
    want = np.cumsum(Gp[0, ::-1].sum(-1), 0)[::-1]  # whole numbers; a state's log-magnitude is at most 8000, good to 8000 eps
    err = 8000 * np.finfo(reals(ctype)).eps * np.abs(Gp).sum() / d
    assert np.abs(host(gm)[0] - want[:, :, None] * np.eye(d)).max() <= err
    assert np.abs(host(gi)[0] - Gp[0].sum(0)).max() <= err


# log-magnitudes where whole numbers are all that is left of them (a state's is their exact sum)
@pytest.mark.parametrize("ctype,at,step", [(np.complex64, 1.0e9, 64.0), (np.complex64, -1.0e9, 128.0), (np.complex128, 1.0e9, 1.0), (np.complex128, -4.0e14, 2.0),
                                           (np.complex128, 5.0e8, 1.0e5)])
@pytest.mark.parametrize("T,chunk", [(2, 0), (24, 8)])
def test_far_log_magnitudes(G, oracle, T, chunk, ctype, at, step):  # noqa: F811
    say(f"scan adjoint, log-magnitudes about {at}, T={T}, {np.dtype(ctype).name}")
    Z = np.full((1, T, 1, 1), step, dtype=ctype)
    S0 = np.full((1, 1, 1), at, dtype=ctype)
    P = (at + step * np.arange(1, T + 1)).astype(ctype).reshape(1, T, 1, 1)
    gm, gi = G.scan_backward(dev(Z), dev(P), dev(np.ones((1, T, 1, 1), dtype=reals(ctype))), dev(S0), chunk_len=chunk)
    # (every ratio is exactly one: a rounding or two a step of what is left of an exponent)
    assert np.allclose(host(gm).ravel(), np.arange(T, 0, -1), rtol=64 * np.finfo(reals(ctype)).eps)
    assert np.allclose(host(gi).ravel(), T, rtol=64 * np.finfo(reals(ctype)).eps)


@pytest.mark.parametrize("d,m", [(4, 4), (30, 30)])
def test_states_far_out_in_double(G, oracle, d, m):  # noqa: F811
    say(f"scan adjoint, states about e^5e8, d={d}")
    ctype, T, at = np.complex128, 20, 5.0e8
    rng = np.random.default_rng(d)
    Z = oracle.to_goom(np.eye(d) + 0.5 / np.sqrt(d) * rng.standard_normal((1, T, d, d)))
    S0 = oracle.to_goom(rng.standard_normal((1, d, m)))
    Gp = rng.standard_normal((1, T, d, m))
    # whole log-magnitudes are exact out there: the same chain, moved
    Z, S0 = (np.rint(Z.real) + 1j * Z.imag).astype(ctype), (np.rint(S0.real) + 1j * S0.imag).astype(ctype)
    far = states(oracle, Z[0], S0[0])[None] + at  # (rounded to 2^-24: what the gradients are of)
    near = (far - at).astype(ctype)
    gm, gi = G.scan_backward(dev(Z), dev(far), dev(Gp), dev((S0 + at).astype(ctype)), chunk_len=8)
    wm, wi, _ = oracle.scan_backward(Z[0], Gp[0], init=S0[0], p=near[0])
    bound = 1000 * 2.0 ** -53 * math.sqrt(T * (d + m))  # as in run(), of sums that are down to a thousandth of their terms here
    assert np.abs(host(gm)[0] - wm).max() <= bound * np.abs(wm).max()
    assert np.abs(host(gi)[0] - wi).max() <= bound * np.abs(wi).max()


# a chunk's product beyond the exponents that the walk carries, in a direction that the states never take
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_product_out_of_range(G, oracle, ctype):  # noqa: F811
    say(f"scan adjoint, a direction out of range, {np.dtype(ctype).name}")
    T, step = 32, 1.0e8
    Z = np.full((1, T, 2, 2), -np.inf, dtype=ctype)
    Z[0, :, 0, 0], Z[0, :, 1, 1], Z[0, :, 1, 0] = step, 0.0, 0.0
    S0 = np.array([[[-np.inf], [0.0]]], dtype=ctype)
    P = np.broadcast_to(S0, (1, T, 2, 1)).copy()
    gm, gi = G.scan_backward(dev(Z), dev(P), dev(np.ones((1, T, 2, 1), dtype=reals(ctype))), dev(S0), chunk_len=8)
    want = np.zeros((T, 2, 2))
    want[:, 1, 1] = np.arange(T, 0, -1)
    assert np.abs(host(gm)[0] - want).max() <= 64 * np.finfo(reals(ctype)).eps * T
    assert np.abs(host(gi)[0, :, 0] - [0.0, T]).max() <= 64 * np.finfo(reals(ctype)).eps * T
