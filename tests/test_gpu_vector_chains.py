"""Chains with a state of one column (recurrences, vector initial states) at the sizes where the matrix-vector kernels can go
wrong: around 16, 32, 64 and 128 rows, one to a few steps, several chunks and groups of chunks, zeros among the entries, one matrix
for all steps; against the oracle, with the tolerances of the parity tests."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, compare, dev, host, lorenz_chain, say, tolerance, with_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu

# (random probes of an entry's sensitivity: two underestimate it tenfold about once in 10^4 entries, and there are many here)
PROBES = 8
SIZES = [1, 3, 8, 15, 16, 17, 24, 31, 32, 33, 47, 48, 63, 64, 65, 96, 100, 127, 128]


def inputs(oracle, seed, batch, T, d, ctype, constant):
    comp = np.float32 if ctype == np.complex64 else np.float64
    A, b = si.recurrence_inputs(si.BASE_SEED + seed, batch, T, d, gain=0.9 if constant else 1.05)
    rng = np.random.default_rng(seed)
    A[rng.random(A.shape) < 0.05] = 0.0  # some zero entries, a zero row and a zero bias
    A[:, T // 2, d // 2] = 0.0
    b[:, T // 3] = 0.0
    if constant:
        A = np.ascontiguousarray(A[:, 0])
    h0 = si.normal_f32(si.BASE_SEED + seed + 1, 9, batch * d).reshape(batch, d)
    return [oracle.to_goom(np.ascontiguousarray(v).astype(comp)) for v in (A, b, h0)]


# chunks of 3 steps make more than 192 of them at T = 600: a grouped carry phase
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("constant", [False, True])
@pytest.mark.parametrize("d", SIZES)
def test_recurrence_sizes(G, oracle, d, ctype, constant):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, batch, chunk in ((1, 3, 0), (2, 1, 1), (5, 2, 2), (61, 2, 0), (61, 2, 7), (600, 1, 3)):
        if T > 500 and d > 33:
            continue
        Az, bz, h0 = inputs(oracle, 300 + d, batch, T, d, ctype, constant)
        say(f"recurrence T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name} constant={constant}")
        rep = (lambda a: np.ascontiguousarray(np.broadcast_to(a[:, None], (batch, T, d, d)))) if constant else (lambda a: a)
        fn = lambda a_, b_, h_: oracle.affine_scan(rep(a_), b_, h0=h_, return_kappa=True)  # noqa: B023
        re, sg, kap, well = with_sensitivity(fn, [Az, bz, h0], comp, nprobe=PROBES)
        got = host(G.affine_scan(dev(Az), dev(bz), dev(h0), chunk_len=chunk, time_invariant=constant))
        compare(got, re, sg, kap, name=f"T{T}d{d}", max_ill_fraction=0.25, well=well)
        # the scaled states belong to the same states: s = +-exp(re - c + 2)
        sc, c = (host(v).astype(np.float64) for v in G.affine_scan_scaled(dev(Az), dev(bz), dev(h0), chunk_len=chunk, time_invariant=constant,
                                                                            want_logscale=True))
        want, cw = oracle.scaled_exp(re + 1j * np.pi * sg)
        top = np.argmax(np.where(np.isfinite(re), re, -np.inf), axis=-1)
        ok = well & (kap <= (2.0 ** 9 if comp == np.float32 else 2.0 ** 30)) & np.take_along_axis(well, top[..., None], axis=-1) & np.isfinite(re)
        tol = tolerance(np.where(np.isfinite(re), re, 0.0), comp) + tolerance(np.where(np.isfinite(cw), cw, 0.0), comp)[..., None]
        assert np.all(np.abs(sc - want)[ok] <= (tol * np.abs(want))[ok])


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", SIZES)
def test_vector_states(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, batch, chunk in ((1, 2, 0), (37, 2, 0), (37, 1, 5), (600, 1, 3)):
        if T > 500 and d > 33:
            continue
        x = si.normal_chain(si.BASE_SEED + 320 + d, batch * T, d).reshape(batch, T, d, d)
        v = si.normal_f32(si.BASE_SEED + 321, 9, batch * d).reshape(batch, d, 1)
        z, u = oracle.to_goom(x.astype(comp)), oracle.to_goom(v.astype(comp))
        say(f"vector state T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name}")
        for q in range(batch):
            fn = lambda m_, i_: oracle.scan(m_, init=i_, return_kappa=True)
            re, sg, kap, well = with_sensitivity(fn, [z[q], u[q]], comp, nprobe=PROBES)
            got = host(G.scan(dev(z), dev(u), chunk_len=chunk))[q]
            compare(got, re, sg, kap, name=f"T{T}d{d}", max_ill_fraction=0.25, well=well)
            last = host(G.reduce(dev(z), dev(u), chunk_len=chunk))[q]
            compare(last, re[-1], sg[-1], kap[-1], name="last", max_ill_fraction=1.0, well=well[-1])
        # one column as a product of its own
        a, b = z[:, 0], u
        fn = lambda a_, b_: oracle.lmme(a_, b_, return_kappa=True)
        re, sg, kap, well = with_sensitivity(fn, [a, b], comp, nprobe=PROBES)
        compare(host(G.lmme(dev(a), dev(b))), re, sg, kap, name="lmme", max_ill_fraction=0.25, well=well)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [5, 48, 100])
def test_magnitudes_far_apart(G, oracle, d, ctype):  # noqa: F811
    """A bias far above and far below the vector's scale, a chain that dies out to zero and starts again, and non-finite input."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    Az, bz, h0 = inputs(oracle, 340 + d, 2, 24, d, ctype, False)
    bz = bz.copy()
    bz[:, 5].real += comp(4000.0)
    bz[:, 11].real -= comp(9000.0)
    Az[:, 15].real = -np.inf  # everything forgotten
    bz[:, 15].real = -np.inf
    bz[:, 16].real -= comp(700.0)
    for chunk in (0, 6):
        re, sg, kap, well = with_sensitivity(lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True), [Az, bz, h0], comp, nprobe=PROBES)
        got = host(G.affine_scan(dev(Az), dev(bz), dev(h0), chunk_len=chunk))
        compare(got, re, sg, kap, name=f"far apart d{d}", max_ill_fraction=0.25, well=well)
        assert np.all(np.isneginf(got.real[:, 15]))
        bad = Az.copy()
        bad[0, 7, 0, 0] = np.nan
        got = host(G.affine_scan(dev(bad), dev(bz), dev(h0), chunk_len=chunk))
        assert np.isnan(got[0, 7].real).any() and np.isfinite(got[1, :15].real).all() and np.isfinite(got[0, :7].real).all()


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("constant", [False, True])
@pytest.mark.parametrize("d", [2, 5, 24, 48, 63, 100, 127])
def test_bias_beside_large_entries_and_cancelled_terms(G, d, constant, ctype):  # noqa: F811
    """A bias is the result where a large entry of A meets a zero (or next to nothing) in the vector; it is dropped only below the last place
    of terms that cancel exactly."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    large, tiny, below, above = (110.0, -200.0, -150.0, -60.0) if comp == np.float32 else (800.0, -1600.0, -900.0, -600.0)
    none, pi = -np.inf, float(comp(np.pi))

    def run(row, h0, bias):
        A = np.full((2, d, d), none, dtype=ctype)
        A[:, 0, 0] = A[:, 1, 1] = 0.0
        A[:, d - 1] = none
        for j, v in row.items():
            A[:, d - 1, j] = v
        b = np.full((1, 2, d), none, dtype=ctype)
        b[0, :, d - 1] = bias
        h = np.full((1, d), none, dtype=ctype)
        for j, v in h0.items():
            h[0, j] = v
        z = A[None, 0] if constant else A[None]
        return host(G.affine_scan(dev(z), dev(b), dev(h), time_invariant=constant))[0, :, d - 1]

    for h0 in ({0: 0.0}, {0: 0.0, d - 1: tiny}):
        got = run({d - 1: large}, h0, 0.0)
        assert got[0] == 0 and abs(got[1].real - large) <= 1e-6 * large, got
    if d > 2:  # h_0 - h_1 with h_0 = h_1 = 1
        for bias, want in ((below, none), (above, above)):
            got = run({0: 0.0, 1: 1j * pi}, {0: 0.0, 1: 0.0}, bias).real
            assert np.all(got == want) or np.allclose(got, want, rtol=1e-6), (bias, got)


@pytest.mark.parametrize("constant", [False, True])
@pytest.mark.parametrize("d", [3, 20, 40, 100])
def test_carries_of_small_rows_and_entries(G, oracle, d, constant):  # noqa: F811
    """Chunk products whose rows lie e^-700 apart on vectors whose entries do (complex128): a row's product with its entry is below the smallest
    double on the matrix's and the vector's powers of two, and e^-50 of the largest result."""
    T, at = 5, [0, d // 2, d - 1]
    A = np.full((1, T, d, d), -np.inf, dtype=np.complex128)
    h0 = np.full((1, d), -np.inf, dtype=np.complex128)
    for i, a, h in zip(at, (0.0, -600.0, -700.0), (-700.0, -150.0, 0.0)):
        A[0, :, i, i] = 0.0
        A[0, : T if constant else 1, i, i] = a
        h0[0, i] = h
    T = 2 if constant else T  # (a third step leaves the vector's own range)
    A, b = np.ascontiguousarray(A[:, :T]), np.full((1, T, d), -np.inf, dtype=np.complex128)
    re, _ = oracle.affine_scan(A, b, h0=h0)
    got = host(G.affine_scan(dev(A[:, 0]) if constant else dev(A), dev(b), dev(h0), chunk_len=1, time_invariant=constant)).real
    assert np.array_equal(np.isneginf(got), np.isneginf(re))
    live = np.isfinite(re)
    assert np.abs(got[live] - re[live]).max() <= 1e-10 * np.abs(re[live]).max(), (got[0][:, at], re[0][:, at])


# (16 and 32: a walk of their own, with one matrix also 64; 96 sequences of 32: the walk sequence by sequence)
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d,batch", [(5, 2), (16, 2), (24, 2), (32, 2), (32, 96), (64, 2), (100, 2)])
def test_scaled_states_that_are_not_numbers(G, oracle, d, batch, ctype):  # noqa: F811
    T, at = 24, 7
    Az, bz, h0 = inputs(oracle, 350 + d, batch, T, d, ctype, False)
    Az[0, at, 0, 0] = bz[0, at, 0] = np.nan
    for chunk, constant in ((0, False), (6, False), (0, True), (4, True)):
        z = np.ascontiguousarray(Az[:, 0]) if constant else Az
        H = host(G.affine_scan(dev(z), dev(bz), dev(h0), chunk_len=chunk, time_invariant=constant)).real
        assert np.isnan(H[0, at]).any() and np.isfinite(H[1]).any(axis=-1).all() and np.isfinite(H[0, at - 1]).any()
        s, c = (host(v) for v in G.affine_scan_scaled(dev(z), dev(bz), dev(h0), chunk_len=chunk, time_invariant=constant, want_logscale=True))
        bad = np.isnan(H).any(axis=-1)
        assert np.array_equal(np.isnan(c), bad) and np.all(np.isnan(s)[np.isnan(H)]) and not np.isnan(s[~bad]).any(), (chunk, constant)


# (the method of test_affine_scan_backward: the oracle on the device's forward states, entries that half-unit perturbations move left out)
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", SIZES)
def test_recurrence_adjoint_sizes(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, batch, chunk, with_h0 in ((1, 3, 0, True), (2, 1, 1, True), (5, 2, 2, False), (61, 2, 0, True), (61, 2, 7, False), (40, 1, 40, True)):
        Az, bz, h0 = inputs(oracle, 360 + d, batch, T, d, ctype, False)
        h0 = h0 if with_h0 else None
        Gh = si.normal_f32(si.BASE_SEED + 361, 10, batch * T * d).reshape(batch, T, d).astype(comp)
        Gh[:, T // 4] = 0.0
        say(f"recurrence adjoint T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name} h0={with_h0}")
        put = lambda z: None if z is None else dev(z)
        Hd = G.affine_scan(dev(Az), dev(bz), put(h0), chunk_len=chunk)
        H = host(Hd)
        got = [None if v is None else host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), put(h0), chunk_len=chunk)]
        want = oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)[:3]
        rel, tiny = (1e-3 if comp == np.float32 else 1e-9), 2 * float(np.finfo(comp).tiny)
        eta = 2.0 ** -24 if comp == np.float32 else 2.0 ** -53
        rng = np.random.default_rng(5)
        sens = [0.0 if w is None else np.zeros_like(w) for w in want]
        for _ in range(PROBES):
            pert = lambda z: None if z is None else (z.astype(np.complex128) + eta * rng.standard_normal(z.shape) * np.where(np.isfinite(z.real), 1.0, 0.0))
            probe = oracle.affine_scan_backward(pert(Az), pert(bz), Gh, h0=pert(h0), h=pert(H))[:3]
            sens = [s if w is None else np.maximum(s, np.abs(p - w)) for s, p, w in zip(sens, probe, want)]
        for name, g, w, s in zip(("A", "bias", "h0"), got, want, sens):
            if w is None or g is None:
                continue
            axes = (-1, -2) if name == "A" else -1
            tol = rel * np.abs(w) + 1e-3 * rel * np.abs(w).max(axis=axes, keepdims=True) + tiny
            well = s <= tol / 16
            assert well.mean() > 0.8, (name, well.mean())
            assert np.all(np.abs(g - w)[well] <= tol[well]), (name, (np.abs(g - w) / tol)[well].max())
        if not with_h0:
            assert np.all(got[0][:, 0] == 0)


def far_apart(oracle, kind, seed, batch, T, d, ctype, spread):
    """A recurrence whose states' entries lie up to e^(2 spread) apart while every gradient is an ordinary number: A and the states in units
    of their own (D_t A_t D_{t-1}^-1, D_t b_t, the units the same at every step or new ones), the matrices dense, triangular, sparse or diagonal."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(seed)
    A, b = rng.standard_normal((batch, T, d, d)) / np.sqrt(d), rng.standard_normal((batch, T, d))
    h0 = rng.standard_normal((batch, d))
    if kind == "triangular":
        A = np.tril(A)
    if kind == "sparse":
        A[rng.random(A.shape) < 0.6] = 0.0
        h0[rng.random(h0.shape) < 0.3] = 0.0
    if kind == "diagonal":
        A = A * np.eye(d) * np.sqrt(d)
        b[...] = 0.0
    unit = rng.uniform(-spread, spread, (batch, T + 1, d)) if kind == "new units" else np.repeat(rng.uniform(-spread, spread, (batch, 1, d)), T + 1, axis=1)
    z = [oracle.to_goom(np.ascontiguousarray(v).astype(comp)) for v in (A, b, h0)]
    z[0].real += (unit[:, 1:, :, None] - unit[:, :-1, None, :]).astype(comp)
    z[1].real += unit[:, 1:].astype(comp)
    z[2].real += unit[:, 0].astype(comp)
    if kind == "diagonal":  # decays at rates of their own
        z[0].real -= np.where(np.eye(d) > 0, rng.uniform(0, spread / T, (batch, 1, d, 1)), 0.0).astype(comp)
    return z


# (one chunk: chunk products hold a matrix on one power of two, and span no more than their type does)
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("kind", ["dense", "triangular", "sparse", "diagonal", "new units"])
@pytest.mark.parametrize("d", [2, 5, 17, 33, 48, 64, 100, 128])
def test_adjoint_of_entries_far_apart(G, oracle, d, kind, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, chunk, spread in ((1, 0, 100.0), (2, 2, 30.0), (12, 12, 100.0), (12, 12, 300.0), (40, 6, 8.0)):
        spread *= 1.0 if comp == np.float32 else 8.0
        Az, bz, h0 = far_apart(oracle, kind, 400 + d + T, 2, T, d, ctype, spread)
        Gh = si.normal_f32(si.BASE_SEED + 401, 10, 2 * T * d).reshape(2, T, d).astype(comp)
        re, sg = oracle.affine_scan(Az, bz, h0=h0)
        H = (re + 1j * np.where(sg, float(comp(np.pi)), 0.0)).astype(ctype)
        say(f"adjoint far apart {kind} T={T} d={d} chunk={chunk} spread={spread} {np.dtype(ctype).name}")
        got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), dev(H), dev(Gh), dev(h0), chunk_len=chunk)]
        want = oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)[:3]
        # Every term is a product of factors that are good to a few units in the last place whatever their size, so a gradient whose terms do
        # not cancel is good to d T units; what half-unit perturbations move further is left out.  Nothing is measured against larger entries.
        # (Half a unit of a double log-magnitude itself: log2(e), one double, times it is the exponent that the device forms.)
        rel = 1e-3 if comp == np.float32 else 1e-9
        eta, tiny = 2.0 ** -24 if comp == np.float32 else 2.0 ** -53, 2 * float(np.finfo(comp).tiny)
        rng = np.random.default_rng(5)
        scale = lambda z: np.where(np.isfinite(z.real), 1.0 if comp == np.float32 else np.maximum(1.0, np.abs(np.where(np.isfinite(z.real), z.real, 0.0))), 0.0)
        pert = lambda z: z.astype(np.complex128) + eta * rng.standard_normal(z.shape) * scale(z)
        sens = [np.zeros_like(w) for w in want]
        for _ in range(PROBES):
            probe = oracle.affine_scan_backward(pert(Az), pert(bz), Gh, h0=pert(h0), h=pert(H))[:3]
            sens = [np.maximum(s, np.abs(p - w)) for s, p, w in zip(sens, probe, want)]
        for name, g, w, s in zip(("A", "bias", "h0"), got, want, sens):
            assert np.isfinite(g).all(), name
            tol = rel * np.abs(w) + tiny
            well = s <= tol / 16
            assert well.mean() > 0.75, (name, well.mean())
            bad = (np.abs(g - w) > tol) & well
            assert not bad.any(), (name, int(bad.sum()), int(well.sum()), (np.abs(g - w) / tol)[well].max())


def test_adjoint_smallest_example_far_apart(G):  # noqa: F811
    """A = 1, no bias, h0 = (1, e^-90): lam_2 = e^90 is no float, and the gradient with respect to A is the identity."""
    for ctype, low in ((np.complex64, -90.0), (np.complex64, -300.0), (np.complex128, -800.0)):
        comp = np.float32 if ctype == np.complex64 else np.float64
        A = np.full((1, 1, 2, 2), -np.inf, dtype=ctype)
        A[0, 0, 0, 0] = A[0, 0, 1, 1] = 0.0
        h = np.array([[0.0, low]], dtype=ctype)
        ga, gb, gh = G.affine_scan_backward(dev(A), dev(np.full((1, 1, 2), -np.inf, dtype=ctype)), dev(h[:, None]), dev(np.ones((1, 1, 2), dtype=comp)), dev(h))
        assert np.allclose(host(ga)[0, 0], np.eye(2), rtol=1e-6, atol=0), host(ga)
        assert np.all(host(gb) == 0) and np.allclose(host(gh), 1.0, rtol=1e-6)
        # an infinite state divides its gradient away (no NaN), and leaves the others'
        h[0, 1] = np.inf
        _, gb, _ = G.affine_scan_backward(dev(A), dev(np.zeros((1, 1, 2), dtype=ctype)), dev(h[:, None]), dev(np.ones((1, 1, 2), dtype=comp)))
        assert np.array_equal(host(gb)[0, 0], [1, 0]), host(gb)


# the batches from which on sequences are walked start to end (no chunks), and one fewer
@pytest.mark.parametrize("ctype,d,line", [(np.complex64, 8, 512), (np.complex64, 24, 192), (np.complex64, 64, 96), (np.complex64, 100, 56),
                                          (np.complex128, 8, 384), (np.complex128, 24, 96), (np.complex128, 48, 48)])
def test_batches_around_the_line(G, oracle, ctype, d, line):  # noqa: F811
    comp, T = np.float32 if ctype == np.complex64 else np.float64, 34
    Az, bz, h0 = inputs(oracle, 390 + d, line, T, d, ctype, False)
    fn = lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [Az, bz, h0], comp)  # (two probes: one entry in 10^4 may be ten times as sensitive as they say)
    for batch in (line, line - 1):
        say(f"batch {batch} T={T} d={d} {np.dtype(ctype).name}")
        A_, b_, h_ = dev(Az[:batch]), dev(bz[:batch]), dev(h0[:batch])
        G.profile_enable(True)
        Hd = G.affine_scan(A_, b_, h_)
        labels = [k for k, _ in G.profile_records()]
        G.profile_enable(False)
        assert (labels == ["affine_single_chunk"]) == (batch == line), labels
        compare(host(Hd), re[:batch], sg[:batch], kap[:batch], name=f"batch {batch}", max_ill_fraction=0.25, well=well[:batch], max_out_fraction=1e-4, hard_factor=10.0)
        H = host(Hd)
        Gh = (si.normal_f32(si.BASE_SEED + 391, 10, batch * T * d).reshape(batch, T, d) * oracle.scaled_exp(H)[0]).astype(comp)
        got = [host(v).astype(np.float64) for v in G.affine_scan_backward(A_, b_, Hd, dev(Gh), h_)]
        want = oracle.affine_scan_backward(Az[:batch], bz[:batch], Gh, h0=h0[:batch], h=H)[:3]
        for name, g, w in zip(("A", "bias", "h0"), got, want):
            assert np.linalg.norm(g - w) <= (1e-3 if comp == np.float32 else 1e-10) * np.linalg.norm(w), (name, np.linalg.norm(g - w) / np.linalg.norm(w))


# more chunks than one chain carries: 192 with one matrix for all steps, 128 in the adjoint pass (there by default too), grouped from there on
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("T,d,batch,chunk,constant", [
    (600, 5, 2, 3, True), (587, 24, 1, 3, True), (400, 16, 2, 2, True), (400, 32, 1, 2, True), (390, 48, 1, 2, True), (400, 64, 1, 2, True), (388, 100, 1, 2, True),
    (195, 17, 2, 1, True), (4096, 5, 1, 0, False), (1500, 24, 1, 0, False), (390, 48, 1, 3, False), (262, 64, 1, 2, False), (264, 100, 1, 2, False), (131, 17, 2, 1, False)])
def test_many_chunks_carried_in_groups(G, oracle, T, d, batch, chunk, constant, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    Az, bz, h0 = inputs(oracle, 380 + d, batch, T, d, ctype, constant)
    say(f"many chunks T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name} constant={constant}")
    rep = np.ascontiguousarray(np.broadcast_to(Az[:, None], (batch, T, d, d))) if constant else Az
    G.profile_enable(True)
    Hd = G.affine_scan(dev(Az), dev(bz), dev(h0), chunk_len=chunk, time_invariant=constant)
    labels = [k for k, _ in G.profile_records()]
    if constant:
        assert labels.count("affine_phase2_carries") == 3, labels
    fn = lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [rep, bz, h0], comp, nprobe=PROBES)
    compare(host(Hd), re, sg, kap, name=f"T{T}d{d}", max_ill_fraction=0.25, well=well)
    # gradients as a layer asks for them, from the scaled states: small entries weigh little
    H = host(Hd)
    Gh = (si.normal_f32(si.BASE_SEED + 381, 10, batch * T * d).reshape(batch, T, d) * oracle.scaled_exp(H)[0]).astype(comp)
    got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), dev(h0), chunk_len=chunk, time_invariant=constant)]
    labels = [k for k, _ in G.profile_records()]
    G.profile_enable(False)
    if not constant and not (comp == np.float32 and d in (16, 32)):
        assert "affine_adjoint_group_products" in labels, labels
    want = (oracle.affine_scan_backward_time_invariant if constant else oracle.affine_scan_backward)(Az, bz, Gh, h0=h0, h=H)[:3]
    # (a norm-wise bound: T steps whose roundings add up; the entries' own bounds are those of the tests above)
    for name, g, w in zip(("A", "bias", "h0"), got, want):
        assert np.linalg.norm(g - w) <= (1e-3 if comp == np.float32 else 1e-10) * np.linalg.norm(w), (name, np.linalg.norm(g - w) / np.linalg.norm(w))


# chunks of 128 (and 64) steps in spans of 16: chains that end within a span, within a chunk, and on both
@pytest.mark.parametrize("T,d,batch,chunk", [(129, 5, 2, 0), (143, 20, 1, 0), (256, 33, 1, 0), (200, 70, 1, 64), (150, 100, 1, 0), (128, 16, 3, 0)])
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_reset_scan_in_spans(G, oracle, T, d, batch, chunk, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(T + d)
    J = (np.eye(d) + 0.1 / np.sqrt(d) * rng.standard_normal((batch, T, d, d))).astype(comp)
    Jz = oracle.to_goom(J)
    say(f"reset scan in spans T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name}")
    states, flags, growth = (host(v) for v in G.scan_reset(dev(Jz), chunk_len=chunk))
    every = chunk or 128
    for q in range(batch):  # the recurrence itself in double, factorised where it is examined
        x, grown = np.eye(d), np.zeros(d)
        rel = np.exp(Jz[q].real.astype(np.float64)) * np.where(Jz[q].imag > 1.5, -1.0, 1.0)
        for t in range(T):
            x = rel[t] @ x
            if (t + 1) % every == 0:
                x, r = np.linalg.qr(x)
                grown += np.log(np.abs(np.diag(r)))
                x *= np.sign(np.diag(r))
                assert flags[q, t] == 1
            got = np.exp(states[q, t].real.astype(np.float64)) * np.where(states[q, t].imag > 1.5, -1.0, 1.0)
            # (a state's float log-magnitudes are rounded once; the double factorisation is good to cond^2 2^-53 of a column)
            assert np.abs(got - x).max() <= (2e-6 if comp == np.float32 else 1e-9) * np.abs(x).max(), (q, t)
        if T % every:
            grown += np.log(np.abs(np.diag(np.linalg.qr(x)[1])))
        assert np.abs(growth[q] - grown).max() <= 1e-8 * max(1.0, np.abs(grown).max())


# an initial state and the policy that looks at the columns, in spans: against the oracle's sequential walk
@pytest.mark.parametrize("T,d,chunk,policy,thr", [(400, 8, 64, 0, 0.9), (300, 33, 64, 0, 0.97), (200, 20, 64, 1, 0.99), (130, 70, 64, 1, 0.99), (300, 12, 0, 1, 0.99)])
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_reset_scan_in_spans_from_an_initial_state(G, oracle, T, d, chunk, policy, thr, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    Jz = oracle.to_goom(lorenz_chain(T, d, 63).astype(comp))
    S0 = oracle.to_goom(si.normal_init(si.BASE_SEED + 63, d, d).astype(comp))
    say(f"reset scan in spans from S0 T={T} d={d} chunk={chunk} policy={policy} {np.dtype(ctype).name}")
    states, flags, growth = (host(v) for v in G.scan_reset(dev(Jz), dev(S0), chunk_len=chunk, policy=policy, cos_threshold=thr))
    re, sg, oflag, ogrowth = oracle.reset_scan(Jz, S0, check_every=chunk or 128, policy=policy, cos_threshold=thr)
    assert np.array_equal(flags, oflag) and oflag.sum() > 0
    got, want = (np.exp(r.astype(np.float64)) * np.where(s, -1.0, 1.0) for r, s in ((states.real, states.imag > 1.5), (re, sg)))
    # (a state's float log-magnitudes are rounded once; the double factorisation is good to cond^2 2^-53 of a column)
    assert np.all(np.abs(got - want).max(axis=(1, 2)) <= (2e-6 if comp == np.float32 else 1e-9) * np.abs(want).max(axis=(1, 2)))
    assert np.abs(growth - ogrowth).max() <= 1e-8 * max(1.0, np.abs(ogrowth).max())
