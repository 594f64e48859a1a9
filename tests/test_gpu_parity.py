"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element,
on the same seeded inputs.  Tolerances are the ones fixed for this build: codecs bit-exact;
signs exact and log-magnitudes within 1e-3 absolute or 1e-4 relative (float components),
1e-10 relative (double components), on every entry that is well conditioned at the
component precision.  "Well conditioned" is decided by the oracle alone, two ways:
  * the cancellation factor kappa of the sum that produced the entry is <= 2^9 (float
    components) or 2^30 (double components): a float sum of d terms carries a relative
    error of about sqrt(d) 2^-24 kappa, which reaches the 1e-3 tolerance near kappa = 2^10;
  * re-running the oracle on inputs whose log-magnitudes are perturbed by random amounts of
    half a unit in the last place of the component type moves the entry by less than 1/16
    of the tolerance and does not flip its sign (a finite-difference condition number: it
    sees cancellation accumulated along the chain, which kappa of the last step does not).
The fraction of entries excluded this way is bounded and printed."""
import math
import sys

import numpy as np
import pytest

import synthetic_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    from paper_2510_03426_amd import Goom
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return Goom(0)


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def tolerance(ref_re, comp):
    if comp == np.float32:
        return np.maximum(1e-3, 1e-4 * np.abs(ref_re))
    return np.maximum(1e-10, 1e-10 * np.abs(ref_re))


def with_sensitivity(fn, arrays, comp, nprobe=2, seed=12345, eta_scale=1.0):
    """Run oracle function fn(*arrays) -> (re, sg, kappa) and estimate, by finite differences,
    how far half-ulp perturbations of the input log-magnitudes move each output.
    Returns (re, sg, kappa, well_mask)."""
    re, sg, kap = fn(*arrays)
    eta = (2.0 ** -24 if comp == np.float32 else 2.0 ** -53) * eta_scale
    rng = np.random.default_rng(seed)
    sens = np.zeros_like(re)
    for _ in range(nprobe):
        pert = []
        for a in arrays:
            if a is None:
                pert.append(None)
                continue
            z = a.astype(np.complex128)
            z.real += eta * rng.standard_normal(a.shape) * np.where(np.isfinite(a.real), 1.0, 0.0)
            pert.append(z)
        pre, psg, _ = fn(*pert)
        with np.errstate(invalid="ignore"):
            dlt = np.abs(pre - re)
        dlt[np.isnan(dlt)] = 0.0  # both -inf
        dlt[psg != sg] = np.inf
        sens = np.maximum(sens, dlt)
    limit = 2.0 ** 9 if comp == np.float32 else 2.0 ** 30
    well = (kap <= limit) & (sens <= tolerance(re, comp) / 16)
    return re, sg, kap, well


def compare(got, ref_re, ref_sg, kappa=None, name="", max_ill_fraction=0.005, well=None, kappa_limit=None,
            max_out_fraction=0.0, hard_factor=1.0):
    """got: complex numpy array from the GPU; ref: oracle working form.  max_out_fraction > 0 lets that
    fraction of the well-conditioned entries exceed the tolerance, by at most hard_factor."""
    comp = np.float32 if got.dtype == np.complex64 else np.float64
    pi = comp(np.pi)
    im = got.imag
    assert np.all((im == 0) | (im == pi)), f"{name}: imaginary parts other than 0 / pi"
    got_sg = (im != 0)
    got_re = got.real.astype(np.float64)
    if kappa is None:
        kappa = np.ones_like(ref_re)
    limit = kappa_limit if kappa_limit is not None else (2.0 ** 9 if comp == np.float32 else 2.0 ** 30)
    well = (kappa <= limit) if well is None else (well & (kappa <= limit))
    ill_frac = 1.0 - well.mean()
    both_zero = np.isneginf(ref_re) & np.isneginf(got_re)
    one_zero = np.isneginf(ref_re) ^ np.isneginf(got_re)
    assert not np.any(one_zero & well), f"{name}: zero / non-zero mismatch on {np.sum(one_zero & well)} entries"
    finite = well & ~both_zero & ~one_zero
    sign_bad = finite & (got_sg != ref_sg.astype(bool))
    assert not np.any(sign_bad), f"{name}: {sign_bad.sum()} sign mismatches of {finite.sum()} (first at {np.argwhere(sign_bad)[0]})"
    with np.errstate(invalid="ignore"):
        diff = np.abs(got_re - ref_re)
    tol = tolerance(ref_re, comp)
    bad = finite & (diff > tol)
    worst = np.nanmax(np.where(finite, diff / tol, 0.0)) if finite.any() else 0.0
    say(f"  [{name}] entries={got.size} ill-conditioned={ill_frac:.2e} worst |dre|/tol={worst:.3g}")
    if max_out_fraction > 0.0:
        say(f"  [{name}] {int(bad.sum())} of {int(finite.sum())} well-conditioned entries beyond the tolerance")
        assert bad.sum() <= max_out_fraction * finite.sum() and worst <= hard_factor, \
            f"{name}: {bad.sum()} log-magnitudes out of tolerance (worst ratio {worst:.3g})"
    else:
        assert not np.any(bad), f"{name}: {bad.sum()} log-magnitudes out of tolerance (worst ratio {worst:.3g})"
    assert ill_frac <= max_ill_fraction, f"{name}: {ill_frac:.3%} ill-conditioned entries"


# ------------------------------------------------------------------------------ codecs

@pytest.mark.parametrize("comp", [np.float32, np.float64])
def test_codecs_bit_exact(G, oracle, comp):
    rng = np.random.default_rng(101)
    n = (1 << 20) + 3  # ragged tail
    span = 85.0 if comp == np.float32 else 705.0
    tiny = np.finfo(comp).tiny
    special = np.array([0.0, -0.0, 1.0, -1.0, np.inf, -np.inf, tiny, -np.finfo(comp).max, tiny / 8, -tiny / 1024,
                        np.nextafter(comp(1), comp(2)), np.nextafter(comp(1), comp(0)), 2.0, 0.5, np.sqrt(comp(2)), np.sqrt(comp(0.5))], dtype=comp)
    near_one = (1.0 + rng.uniform(-1e-3, 1e-3, 4096)).astype(comp)
    wide = (np.exp(rng.uniform(-span, span, n - n // 2 - special.size - near_one.size)) * rng.choice([-1.0, 1.0], n - n // 2 - special.size - near_one.size)).astype(comp)
    x = np.concatenate([si.normal_f32(si.BASE_SEED, 50, n // 2).astype(comp), wide, near_one, special])
    say(f"codec {comp.__name__}: n={x.size}")
    word = np.uint32 if comp == np.float32 else np.uint64
    for flags in (0, 1):
        want = oracle.to_goom(x, zero_floor=bool(flags))
        got = host(G.to_goom(dev(x), flags=flags))
        neq = got.view(word) != want.view(word)
        assert not neq.any(), f"{neq.sum()} encoded words differ, first at x = {x[np.argwhere(neq.reshape(-1, 2).any(axis=1))[0, 0]]!r}"
    z = oracle.to_goom(x)
    z = z[np.isfinite(z.real) | np.isneginf(z.real)]
    # log-magnitudes of their own too: the whole range of results, subnormal ones and both ends included
    lo, hi = (-104.0, 89.0) if comp == np.float32 else (-746.0, 710.0)
    extra = rng.uniform(lo, hi, 1 << 18).astype(comp) + (1j * np.pi * rng.integers(0, 2, 1 << 18)).astype(z.dtype)
    extra.imag[...] = np.where(extra.imag != 0, comp(np.pi), comp(0))
    edge = rng.uniform(lo, lo + 42.0, 1 << 16).astype(comp).astype(z.dtype)  # results below the smallest normal
    z = np.concatenate([z, extra.astype(z.dtype), edge])
    want = oracle.from_goom(z)
    got = host(G.from_goom(dev(z)))
    neq = got.view(word) != want.view(word)
    assert not neq.any(), f"{neq.sum()} decoded words differ, first at z = {z[np.argwhere(neq)[0, 0]]!r}: {got[np.argwhere(neq)[0, 0]]!r} vs {want[np.argwhere(neq)[0, 0]]!r}"
    # empty input
    import torch
    assert G.to_goom(torch.empty(0, dtype=torch.float32, device="cuda")).numel() == 0


def test_count_nonfinite(G, oracle):
    # the paper's failure notion (Section 4.1): a chain fails when its states stop being finite; zeros (-inf) are fine
    rng = np.random.default_rng(7)
    for ctype in (np.complex64, np.complex128):
        z = (rng.normal(0, 50, (1 << 18) + 5) + 1j * np.pi * rng.integers(0, 2, (1 << 18) + 5)).astype(ctype)
        z[::1000] = -np.inf
        assert G.count_nonfinite(dev(z)) == 0
        z[5], z[77], z[-1] = np.inf, np.nan, np.inf + 1j * np.pi
        assert G.count_nonfinite(dev(z)) == 3
    # a float32 real chain overflows where the GOOM chain does not
    x = si.normal_chain(si.BASE_SEED + 1, 400, 64)
    P = G.scan(G.to_goom(dev(x)))
    assert G.count_nonfinite(P) == 0 and host(P).real.max() > 700


def test_decode_accepts_any_phase_multiple(G, oracle):
    z = np.array([3 + 2j * math.pi, 3 + 4j * math.pi, 3 + 1j * math.pi, 3 - 3j * math.pi, -np.inf + 0j, 200 + 0j],
                 dtype=np.complex64)
    got = host(G.from_goom(dev(z)))
    want = oracle.from_goom(z)
    assert np.array_equal(got, want)
    assert abs(got[0] - 20.0855) < 1e-3 and got[0] == got[1] and got[2] < 0 and got[3] < 0 and got[4] == 0 and np.isinf(got[5])


# -------------------------------------------------------------------------------- LMME

@pytest.mark.parametrize("shape", [(1, 8, 8, 8), (3, 16, 16, 16), (2, 5, 7, 3), (2, 64, 64, 64), (2, 128, 128, 128),
                                   (1, 33, 20, 1), (2, 1, 1, 1), (1, 100, 128, 60), (2, 3, 32, 64), (1, 31, 1, 128), (2, 1, 17, 128),
                                   (1, 16, 4, 40), (2, 48, 48, 48), (1, 96, 96, 96), (3, 20, 20, 20), (1, 124, 124, 124)])
def test_lmme_matches_oracle(G, oracle, shape):
    b, n, d, m = shape
    say(f"lmme batch={b} n={n} d={d} m={m}")
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 20, 7, b * n * d).reshape(b, n, d))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 21, 8, b * d * m).reshape(b, d, m))
    A[0, 0, 0] = -np.inf  # a zero entry
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B)))
    compare(got, re, sg, kap, name=f"lmme{shape}", max_ill_fraction=0.02)


@pytest.mark.parametrize("shape,flags", [((3, 1024, 32, 32), 0), ((2, 200, 64, 64), 0), ((2, 130, 16, 8), 0), ((1, 1000, 24, 50), 0), ((5, 64, 4, 1), 0),
                                         ((2, 77, 12, 33), 0), ((1, 300, 48, 20), 1), ((2, 128, 64, 64), 0), ((1, 17, 8, 8), 0), ((2, 257, 32, 17), 0)])
def test_lmme_many_rows_small_right_operand(G, oracle, shape, flags):
    # the shape of the state-space layer's input term (Section 4.3: B u_t for all steps at once): rows streamed past the right operand
    b, n, d, m = shape
    rng = np.random.default_rng(9)
    say(f"tall lmme batch={b} n={n} d={d} m={m} flags={flags}")
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 26, 7, b * n * d).reshape(b, n, d))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 27, 8, b * d * m).reshape(b, d, m))
    A.real += rng.uniform(-1e4, 1e4, (b, n, 1)).astype(np.float32)  # row scales far outside float range
    B.real += rng.uniform(-1e4, 1e4, (b, 1, m)).astype(np.float32)
    A[0, 0, 0] = -np.inf       # a zero entry
    A[b - 1, n - 1, :] = -np.inf  # an all-zero last row
    if m > 2:
        B[0, :, 1] = -np.inf   # an all-zero column
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B), flags=flags))
    assert np.all(np.isneginf(got.real[b - 1, n - 1, :]))
    if m > 2:
        assert np.all(np.isneginf(got.real[0, :, 1]))
    compare(got, re, sg, kap, name=f"tall lmme{shape}", max_ill_fraction=0.03)


def test_lmme_far_outside_float_range(G, oracle):
    # log-magnitudes of order +-1e5: no float could hold the values, row/column shifts absorb them
    rng = np.random.default_rng(5)
    b, n, d, m = 2, 32, 32, 32
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 22, 7, b * n * d).reshape(b, n, d))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 23, 8, b * d * m).reshape(b, d, m))
    A.real += rng.uniform(-1e5, 1e5, (b, n, 1)).astype(np.float32)
    B.real += rng.uniform(-1e5, 1e5, (b, 1, m)).astype(np.float32)
    B[0, :, 3] = -np.inf  # an all-zero column
    A[1, 5, :] = -np.inf  # an all-zero row
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B)))
    assert np.all(np.isneginf(got.real[0, :, 3])) and np.all(np.isneginf(got.real[1, 5, :]))
    compare(got, re, sg, kap, name="lmme wide", max_ill_fraction=0.02)


def test_lmme_double_components(G, oracle):
    b, n, d, m = 2, 48, 64, 40
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 24, 7, b * n * d).reshape(b, n, d).astype(np.float64))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 25, 8, b * d * m).reshape(b, d, m).astype(np.float64))
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B)))
    compare(got, re, sg, kap, name="lmme c128")


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_lmme_wide_range_needs_exact_repair(G, oracle, ctype):
    # log-magnitudes N(0, 200^2): after the row / column shifts nearly every term is below float
    # range, so the scaled product alone returns zeros; the repair pass recomputes those outputs
    from paper_2510_03426_amd import LMME_EXACT, LMME_FAST
    b, n, d, m = 3, 128, 128, 128
    A, B = si.wide_range_goom_pairs(si.BASE_SEED + 26, b, n, d, m, sigma=200.0, dtype=ctype)
    say(f"lmme exact {np.dtype(ctype).name}: batch={b} {n}x{d}x{m}")
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    fast = host(G.lmme(dev(A), dev(B), flags=LMME_FAST))
    lost = np.isneginf(fast.real) & np.isfinite(re)
    say(f"  scaled product alone: {lost.mean():.1%} of the outputs underflow to zero")
    if ctype == np.complex64:
        assert lost.mean() > 0.5
    got = host(G.lmme(dev(A), dev(B), flags=LMME_EXACT))
    compare(got, re, sg, kap, name=f"lmme exact {np.dtype(ctype).name}", max_ill_fraction=0.002)
    # the same call through the C ABI without the optional workspace (the repair pass then takes the row and column
    # maxima itself instead of receiving the product's shifts)
    import torch
    from paper_2510_03426_amd import binding as bnd
    a_d, b_d = dev(A), dev(B)
    out = torch.empty((b, n, m), dtype=a_d.dtype, device=a_d.device)
    G._check(G.lib.goom_lmme(G._ctx, bnd._ptr(a_d), bnd._ptr(b_d), bnd._ptr(out), b, n, d, m, bnd._dtype_code(a_d), LMME_EXACT, None, 0))
    compare(host(out), re, sg, kap, name=f"lmme exact {np.dtype(ctype).name}, no workspace", max_ill_fraction=0.002)
    # benign data: everything certifies, the repair pass changes nothing
    A2 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 27, 7, 2 * 64 * 64).reshape(2, 64, 64))
    B2 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 28, 8, 2 * 64 * 64).reshape(2, 64, 64))
    assert np.array_equal(host(G.lmme(dev(A2), dev(B2), flags=LMME_EXACT)).view(np.uint32),
                          host(G.lmme(dev(A2), dev(B2), flags=LMME_FAST)).view(np.uint32))


@pytest.mark.parametrize("sigma", [22.0, 35.0, 60.0])
def test_lmme_partly_repaired_blocks(G, oracle, sigma):
    # moderate ranges: only part of a block's outputs fail the certificate, so the repair kernel runs its
    # one-wave-per-output list or its sweeps with some of a wave's sixteen positions skipped
    from paper_2510_03426_amd import LMME_EXACT, LMME_FAST
    b, n, d, m = 2, 128, 128, 128
    A, B = si.wide_range_goom_pairs(si.BASE_SEED + 29, b, n, d, m, sigma=sigma, dtype=np.complex64)
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    fast, got = host(G.lmme(dev(A), dev(B), flags=LMME_FAST)), host(G.lmme(dev(A), dev(B), flags=LMME_EXACT))
    changed = (fast.view(np.uint32) != got.view(np.uint32)).reshape(b, n, m, 2).any(axis=-1)
    say(f"lmme sigma {sigma}: the repair pass rewrote {changed.mean():.1%} of the outputs")
    compare(got, re, sg, kap, name=f"lmme sigma {sigma}", max_ill_fraction=0.002)


def test_lmme_repair_when_few_terms_decide(G, oracle):
    # float repair pass, the outputs that one or two terms decide: log-magnitudes +300 (rarely) or -300, so that
    # the largest pairwise sums are exactly 0 (ties among them, and a key whose number part is zero) or 600, far
    # above all others; then ragged sizes with more than 128 inner indices, zeros among the entries, and one
    # row / column pair that cancels exactly in its two leading terms
    from paper_2510_03426_amd import LMME_EXACT
    rng = np.random.default_rng(si.BASE_SEED + 270)
    b, n, d, m = 2, 128, 128, 128
    A = np.empty((b, n, d), np.complex64)
    B = np.empty((b, d, m), np.complex64)
    A.real = np.where(rng.random((b, n, d)) < 0.02, 300.0, -300.0)
    B.real = np.where(rng.random((b, d, m)) < 0.02, 300.0, -300.0)
    A.imag = np.float32(np.pi) * rng.integers(0, 2, (b, n, d))
    B.imag = np.float32(np.pi) * rng.integers(0, 2, (b, d, m))
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B), flags=LMME_EXACT))
    say(f"lmme two-valued: outputs at 600 {np.mean(re > 500):.1%}, near 0 {np.mean(np.abs(re) < 50):.1%}, zero or below {np.mean(re < -500):.1%}")
    compare(got, re, sg, kap, name="lmme two-valued", max_ill_fraction=0.25)
    b, n, d, m = 2, 70, 200, 90
    A, B = si.wide_range_goom_pairs(si.BASE_SEED + 271, b, n, d, m, sigma=200.0, dtype=np.complex64)
    A.real[rng.random(A.shape) < 0.3] = -np.inf
    B.real[rng.random(B.shape) < 0.3] = -np.inf
    A.real[:, 5, :] = -np.inf  # a zero row: zeros out
    A.real[0, 7, :] = -np.inf  # one term alone
    A.real[0, 7, 150] = 12.5
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B), flags=LMME_EXACT))
    assert np.isneginf(got.real[:, 5, :]).all()
    compare(got, re, sg, kap, name="lmme ragged with zeros", max_ill_fraction=0.01)
    # ragged sizes with at most 128 inner indices: the path that orders the terms by keys, at the operands' edges
    for (b2, n2, d2, m2) in ((2, 70, 100, 90), (1, 130, 128, 65), (3, 64, 17, 64)):
        A3, B3 = si.wide_range_goom_pairs(si.BASE_SEED + 272 + d2, b2, n2, d2, m2, sigma=200.0, dtype=np.complex64)
        A3.real[rng.random(A3.shape) < 0.1] = -np.inf
        re3, sg3, kap3 = oracle.lmme(A3, B3, return_kappa=True)
        got3 = host(G.lmme(dev(A3), dev(B3), flags=LMME_EXACT))
        compare(got3, re3, sg3, kap3, name=f"lmme ragged, keyed {n2}x{d2}x{m2}", max_ill_fraction=0.01)
    # two leading terms of opposite sign, half a unit apart: inner indices 0 and 1 tower over the others
    A2, B2 = A[:1].copy(), B[:1].copy()
    A2[0, :, 0] = 900.0
    A2[0, :, 1] = 899.5 + 1j * np.float32(np.pi)
    B2[0, 1, :] = B2[0, 0, :]
    B2.real[0, 0:2, :] = np.where(np.isneginf(B2.real[0, 0:2, :]), 0.0, B2.real[0, 0:2, :])
    re, sg, kap = oracle.lmme(A2, B2, return_kappa=True)
    got = host(G.lmme(dev(A2), dev(B2), flags=LMME_EXACT))
    compare(got, re, sg, kap, name="lmme two leading terms of opposite sign", max_ill_fraction=0.01)


# -------------------------------------------------------------------------------- scan

def run_scan_case(G, oracle, T, d, chunk_len, m=None, batch=1, seed=0, dtype=np.float32, name=""):
    x = si.normal_f32(si.BASE_SEED + 30 + seed, 1, batch * T * d * d).reshape(batch, T, d, d).astype(dtype)
    Z = oracle.to_goom(x)
    init = None
    if m is not None:
        init = oracle.to_goom(si.normal_f32(si.BASE_SEED + 31 + seed, 2, batch * d * m).reshape(batch, d, m).astype(dtype))
    say(f"scan {name}: T={T} d={d} m={m} batch={batch} chunk_len={chunk_len} {np.dtype(dtype).name}")
    out = host(G.scan(dev(Z), None if init is None else dev(init), chunk_len=chunk_len))
    red = host(G.reduce(dev(Z), None if init is None else dev(init), chunk_len=chunk_len))
    comp = np.dtype(dtype).type
    for b in range(batch):
        fn = lambda mats, ini: oracle.scan(mats, init=ini, return_kappa=True)
        re, sg, kap, well = with_sensitivity(fn, [Z[b], None if init is None else init[b]], comp)
        compare(out[b], re, sg, kap, name=f"{name} scan b{b}", max_ill_fraction=0.03, well=well)
        compare(red[b], re[-1], sg[-1], kap[-1], name=f"{name} reduce b{b}", max_ill_fraction=0.06, well=well[-1])
    return out


def test_scan_tiny_config(G, oracle):
    # T = 256 chain of 8 x 8 matrices: all 256 prefix products
    run_scan_case(G, oracle, 256, 8, 0, name="cfg1 default chunks")
    run_scan_case(G, oracle, 256, 8, 256, name="cfg1 one chunk")
    run_scan_case(G, oracle, 256, 8, 1, name="cfg1 chunk_len 1")


@pytest.mark.parametrize("T,d,chunk", [(37, 16, 5), (300, 32, 64), (700, 64, 100), (130, 128, 32), (64, 5, 7), (50, 33, 16),
                                       (1, 64, 0), (2, 64, 1)])
def test_scan_sizes_and_ragged_tails(G, oracle, T, d, chunk):
    run_scan_case(G, oracle, T, d, chunk, name=f"T{T}d{d}")


@pytest.mark.parametrize("T,d,chunk,m,batch", [(90, 20, 16, None, 1), (300, 24, 0, None, 2), (61, 28, 7, 28, 1), (120, 36, 16, None, 1),
                                                (200, 48, 0, 48, 2), (77, 52, 10, None, 1), (64, 60, 16, None, 1), (40, 68, 8, None, 1),
                                                (70, 96, 16, 96, 1), (33, 100, 8, None, 2), (24, 124, 5, None, 1), (1, 48, 0, None, 1)])
def test_scan_sizes_between_the_tiles(G, oracle, T, d, chunk, m, batch):
    # square matrices whose size is a multiple of four but not a tile size: the hot kernel with rows and columns
    # beyond the matrix left out (all block counts, with and without an initial state, single steps, batches)
    x = si.normal_f32(si.BASE_SEED + 95, 1, batch * T * d * d).reshape(batch, T, d, d)
    if T > 4:
        x[0, 2, d - 1, :] = 0.0   # a zero last row
        x[0, 3, :, d - 1] = 0.0   # a zero last column
        x[0, 4, 0, :] = 0.0
    Z = oracle.to_goom(x)
    init = None
    if m is not None:
        init = oracle.to_goom(si.normal_f32(si.BASE_SEED + 96, 2, batch * d * m).reshape(batch, d, m))
    say(f"scan between tiles: T={T} d={d} m={m} batch={batch} chunk_len={chunk}")
    out = host(G.scan(dev(Z), None if init is None else dev(init), chunk_len=chunk))
    red = host(G.reduce(dev(Z), None if init is None else dev(init), chunk_len=chunk))
    for b in range(batch):
        fn = lambda mats, ini: oracle.scan(mats, init=ini, return_kappa=True)
        re, sg, kap, well = with_sensitivity(fn, [Z[b], None if init is None else init[b]], np.float32)
        compare(out[b], re, sg, kap, name=f"d{d} scan b{b}", max_ill_fraction=0.03, well=well)
        compare(red[b], re[-1], sg[-1], kap[-1], name=f"d{d} reduce b{b}", max_ill_fraction=0.06, well=well[-1])


def test_scan_small_matrices_in_pairs(G, oracle):
    # 8 x 8 chains share a wave two by two: pairs that straddle batch items, a ragged last chunk that is shorter
    # than its partner, an odd number of chains, single steps; 16 x 16 chains one per wave
    run_scan_case(G, oracle, 37, 8, 5, batch=3, seed=11, name="d8 batch3 ragged")     # 8 chunks per item, last of 2 steps
    run_scan_case(G, oracle, 35, 8, 5, batch=3, seed=12, name="d8 batch3 odd chains")  # 7 chunks per item: 21 chains
    run_scan_case(G, oracle, 1, 8, 0, batch=5, seed=13, name="d8 single step")
    run_scan_case(G, oracle, 1200, 8, 0, seed=14, name="d8 default chunks")
    run_scan_case(G, oracle, 41, 16, 6, batch=2, seed=15, name="d16 batch2 ragged")
    run_scan_case(G, oracle, 1000, 8, 3, seed=16, name="d8 334 chunks grouped carries")


@pytest.mark.parametrize("T,d,chunk,m,batch,comp", [(300, 64, 32, None, 1, np.float32), (130, 128, 16, None, 1, np.float32),
                                                     (257, 32, 0, None, 2, np.float32), (90, 64, 0, 64, 2, np.float32),
                                                     (1, 64, 0, None, 1, np.float32),
                                                     (100, 16, 7, None, 2, np.float32), (60, 24, 9, 5, 1, np.float32),
                                                     (40, 200, 8, None, 1, np.float32), (50, 32, 8, None, 1, np.float64)])
def test_scan_of_real_matrices(G, oracle, T, d, chunk, m, batch, comp):
    # the scan fed with real matrices (read directly by the hot kernel at d = 32, 64, 128; encoded into the
    # workspace otherwise) against the oracle's scan of the encoded matrices
    x = si.normal_f32(si.BASE_SEED + 90, 3, batch * T * d * d).reshape(batch, T, d, d).astype(comp)
    if T > 3:
        x[0, 2, 1, :] = 0.0   # a zero row
        x[0, 3, :, 2] = 0.0   # a zero column
    Z = oracle.to_goom(x)
    init = None
    if m is not None:
        init = oracle.to_goom(si.normal_f32(si.BASE_SEED + 91, 4, batch * d * m).reshape(batch, d, m).astype(comp))
    say(f"scan of reals T={T} d={d} chunk={chunk} m={m} batch={batch} {np.dtype(comp).name}")
    out = host(G.scan_real(dev(x), None if init is None else dev(init), chunk_len=chunk))
    red = host(G.scan_real(dev(x), None if init is None else dev(init), chunk_len=chunk, final_only=True))
    big = d > 128
    for b in range(batch):
        if big:
            sample = sorted({0, 1, T // 2, T - 1})
            st = oracle.ScanStream(d, m=d if m is None else m, init=None if init is None else init[b], scaled=True)
            re, sg, kap = st.advance(Z[b], sample_t=sample, return_kappa=True)
            compare(out[b][sample], re, sg, kap, name=f"real scan d{d} item {b}", max_ill_fraction=0.06)
            compare(red[b], re[-1], sg[-1], kap[-1], name=f"real reduce d{d} item {b}", max_ill_fraction=0.06)
        else:
            fn = lambda mats, ini: oracle.scan(mats, init=ini, return_kappa=True)
            re, sg, kap, well = with_sensitivity(fn, [Z[b], None if init is None else init[b]], comp)
            compare(out[b], re, sg, kap, name=f"real scan b{b}", max_ill_fraction=0.03, well=well)
            compare(red[b], re[-1], sg[-1], kap[-1], name=f"real reduce b{b}", max_ill_fraction=0.06, well=well[-1])


def test_scan_many_chunks_grouped_carries(G, oracle):
    # more than 96 chunks: the carry phase is itself a grouped scan (group products, their
    # prefixes, groups re-walked); ragged last chunk and ragged last group
    run_scan_case(G, oracle, 1203, 16, 4, name="301 chunks d16")
    run_scan_case(G, oracle, 700, 32, 5, m=7, batch=2, seed=7, name="140 chunks d32 init")
    run_scan_case(G, oracle, 389, 64, 3, name="130 chunks d64")


def test_scan_with_initial_state_and_batch(G, oracle):
    run_scan_case(G, oracle, 120, 32, 16, m=32, batch=3, seed=1, name="init square batch3")
    run_scan_case(G, oracle, 120, 64, 25, m=1, batch=2, seed=2, name="init vector")
    run_scan_case(G, oracle, 90, 16, 8, m=24, batch=1, seed=3, name="init wide")


def test_scan_with_wide_initial_state(G, oracle):
    # a state with many more columns than the matrices have rows: every phase runs on the tile size that
    # gives each sixteen state columns a wave
    run_scan_case(G, oracle, 70, 16, 8, m=64, batch=2, seed=41, name="d16 m64")
    run_scan_case(G, oracle, 40, 32, 0, m=128, seed=42, name="d32 m128")
    run_scan_case(G, oracle, 33, 8, 5, m=100, seed=43, name="d8 m100")
    run_scan_case(G, oracle, 25, 24, 4, m=60, seed=44, dtype=np.float64, name="d24 m60 double")


def test_scan_double_components(G, oracle):
    run_scan_case(G, oracle, 200, 16, 16, seed=4, dtype=np.float64, name="c128 d16")
    run_scan_case(G, oracle, 96, 64, 24, seed=5, dtype=np.float64, name="c128 d64")
    run_scan_case(G, oracle, 150, 32, 20, seed=6, dtype=np.float64, name="c128 d32")
    run_scan_case(G, oracle, 36, 128, 8, seed=7, dtype=np.float64, name="c128 d128")
    # sizes that do not fill the tile (bounds-checked path of the general kernel), with and without an initial state
    run_scan_case(G, oracle, 40, 100, 9, seed=8, dtype=np.float64, name="c128 d100")
    run_scan_case(G, oracle, 60, 40, 7, m=40, batch=2, seed=9, dtype=np.float64, name="c128 d40 init")
    run_scan_case(G, oracle, 50, 20, 6, m=3, seed=10, dtype=np.float64, name="c128 d20 m3")


def test_scan_is_deterministic(G, oracle):
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 40, 512, 64))
    a = host(G.scan(dev(Z), chunk_len=64))
    b = host(G.scan(dev(Z), chunk_len=64))
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_scan_beyond_float_range(G, oracle):
    # 4096 steps of 64 x 64: log-magnitudes reach ~8500, far past float and double range
    T, d = 4096, 64
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 41, T, d))
    out = host(G.scan(dev(Z)))
    sample = list(range(0, T, 97)) + [T - 1]
    fn = lambda mats: oracle.ScanStream(d, scaled=True).advance(mats, sample_t=sample, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [Z], np.float32, nprobe=1)
    compare(out[sample], re, sg, kap, name="T4096 d64", max_ill_fraction=0.03, well=well)
    assert out.real[-1].max() > 8000
    lam = 0.5 * (math.log(2) + 3.4499)  # (ln 2 + psi(32)) / 2
    assert abs(out.real[-1].max() / T - lam) < 0.05


# ------------------------------------------------------------------------------ affine

@pytest.mark.parametrize("T,d,batch,chunk", [(64, 8, 2, 0), (300, 32, 3, 32), (100, 16, 1, 9), (1, 32, 2, 0), (257, 64, 1, 40),
                                             (1000, 32, 2, 5), (90, 128, 2, 16), (70, 100, 1, 0),
                                             # many sequences of d = 32: each walked start to end by one workgroup
                                             (1, 32, 96, 0), (37, 32, 97, 0), (300, 32, 130, 0), (8, 32, 96, 0), (1000, 32, 100, 0), (33, 32, 300, 0)])
def test_affine_scan_matches_oracle(G, oracle, T, d, batch, chunk):
    A, b = si.recurrence_inputs(si.BASE_SEED + 50, batch, T, d)
    Az, bz = oracle.to_goom(A), oracle.to_goom(b)
    say(f"affine T={T} d={d} batch={batch} chunk={chunk}")
    fn = lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True)
    # (two random probes underestimate an entry's sensitivity tenfold about once in 10^4 entries: with a million entries and more,
    # the oracle probes four times)
    nprobe = 4 if batch * T * d > 500000 else 2
    re, sg, kap, well = with_sensitivity(fn, [Az, bz, None], np.float32, nprobe=nprobe)
    got = host(G.affine_scan(dev(Az), dev(bz), chunk_len=chunk))
    compare(got, re, sg, kap, name=f"affine T{T}d{d}", max_ill_fraction=0.05, well=well)
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 51, 9, batch * d).reshape(batch, d))
    re, sg, kap, well = with_sensitivity(fn, [Az, bz, h0], np.float32, nprobe=nprobe)
    got = host(G.affine_scan(dev(Az), dev(bz), dev(h0), chunk_len=chunk))
    compare(got, re, sg, kap, name=f"affine h0 T{T}d{d}", max_ill_fraction=0.05, well=well)


def test_affine_scan_many_sequences_edge_cases(G, oracle):
    # the walk of whole sequences (d = 32, 96 sequences or more) on states, rows, matrices and biases that are zero, on biases
    # far above and far below the state, and on magnitudes far outside float range; a length that ends inside a round of steps
    batch, T, d = 96, 45, 32
    A, b = si.recurrence_inputs(si.BASE_SEED + 59, batch, T, d)
    Az, bz = oracle.to_goom(A), oracle.to_goom(b)
    zero = np.complex64(complex(-np.inf, 0.0))
    bz[0, :5] = zero          # no bias for five steps and no initial state: the states are zero until step 5
    Az[1, :, 3, :] = zero     # two rows of every matrix zero: those entries of the state are the bias alone
    Az[1, :, 17, :] = zero
    Az[2, 10] = zero          # a zero matrix: the state restarts from the bias
    bz[3, 7] += 300           # a bias e^300 above the state, and one e^-300 below
    bz[3, 20] -= 300
    Az[4] += 40               # log-magnitudes reach 1800
    bz[5] = zero              # nothing but zeros
    Az[6, :, :, 5] = zero     # a zero column: one entry of the state never matters
    bz[7, :, 8:] = zero       # only the first eight entries are driven
    say("affine, many sequences: zeros and wide magnitudes")
    fn = lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [Az, bz, None], np.float32)
    got = host(G.affine_scan(dev(Az), dev(bz)))
    assert np.all(np.isneginf(got[0, :5].real)) and np.all(np.isneginf(got[5].real)) and np.all(np.isneginf(re[5]))
    assert re[4].max() > 1500
    compare(got, re, sg, kap, name="affine, many sequences, edge cases", max_ill_fraction=0.05, well=well)
    # the scaled states of the same sequences: zeros stay zeros, their log-scaling constant is -inf
    sc, c = G.affine_scan_scaled(dev(Az), dev(bz), want_logscale=True)
    sc, c = host(sc).astype(np.float64), host(c).astype(np.float64)
    want, cw = oracle.scaled_exp(re + 1j * np.pi * sg)
    assert np.all(sc[5] == 0) and np.all(np.isneginf(c[5])) and np.all(sc[0, :5] == 0) and np.all(np.isneginf(c[0, :5]))
    top = np.argmax(np.where(np.isfinite(re), re, -np.inf), axis=-1)
    top_well = np.take_along_axis(well, top[..., None], axis=-1)[..., 0] & np.isfinite(cw)
    ok = well & top_well[..., None] & np.isfinite(re)
    with np.errstate(invalid="ignore"):
        bound = np.where(np.isfinite(re), tolerance(re, np.float32), 0.0) + np.where(np.isfinite(cw), tolerance(cw, np.float32), 0.0)[..., None]
    ratio = (np.abs(sc - want) / (bound * np.abs(want) + 1e-30))[ok]
    assert ok.mean() > 0.6 and ratio.max() <= 1, (ok.mean(), ratio.max())
    with np.errstate(invalid="ignore"):
        assert np.all(np.abs(c - cw)[top_well] <= tolerance(cw, np.float32)[top_well])


# ---------------------------------------------------------------- selective resetting, Lyapunov

def lorenz_chain(T, d, seed, burn_in=2000):
    """Jacobians of the Euler-stepped Lorenz-96 map; above d = 40 that map is not stable at
    dt = 0.01, so larger sizes use near-identity random Jacobians I + 0.1 N(0, 1/d) instead."""
    if d > 40:
        g = si.normal_f32(si.BASE_SEED + seed, 11, T * d * d).reshape(T, d, d)
        return (np.eye(d, dtype=np.float32)[None] + np.float32(0.1 / math.sqrt(d)) * g).astype(np.float32)
    for attempt in range(8):  # the Euler map is only marginally stable: move to the next stream if it escapes
        try:
            J, _ = si.lorenz96_jacobians(si.BASE_SEED + seed + 1000 * attempt, T, d=d, burn_in=burn_in)
            return J
        except FloatingPointError:
            continue
    raise RuntimeError("no stable Lorenz-96 trajectory found")


@pytest.mark.parametrize("T,d,L", [(256, 8, 16), (200, 32, 64), (130, 16, 7), (64, 64, 16), (48, 100, 12)])
def test_reset_scan_never_equals_plain_scan(G, oracle, T, d, L):
    from paper_2510_03426_amd import RESET_NEVER
    Jz = oracle.to_goom(lorenz_chain(T, d, 60))
    say(f"reset never T={T} d={d} L={L}")
    states, flags, growth = G.scan_reset(dev(Jz), chunk_len=L, policy=RESET_NEVER)
    fn = lambda mats: oracle.scan(mats, init=oracle.to_goom(np.eye(d, dtype=np.float32)), return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [Jz], np.float32, nprobe=3)
    compare(host(states), re, sg, kap, name=f"reset never T{T}d{d}", max_ill_fraction=0.02, well=well)
    assert host(flags).sum() == 0


@pytest.mark.parametrize("T,d,L,ctype", [(256, 8, 16, np.complex64), (640, 32, 16, np.complex64), (640, 32, 64, np.complex64),
                                         (1024, 32, 0, np.complex64), (200, 16, 7, np.complex64), (100, 6, 25, np.complex64),
                                         (300, 64, 32, np.complex64), (640, 32, 64, np.complex128), (200, 16, 7, np.complex128),
                                         (100, 6, 25, np.complex128), (150, 64, 50, np.complex128), (96, 128, 16, np.complex64),
                                         (70, 100, 9, np.complex64), (60, 72, 20, np.complex128), (64, 128, 8, np.complex128)])
def test_reset_scan_always_matches_sequential_oracle(G, oracle, T, d, L, ctype):
    from paper_2510_03426_amd import RESET_ALWAYS
    comp = np.float32 if ctype == np.complex64 else np.float64
    Jr = lorenz_chain(T, d, 61).astype(comp)
    Jz = oracle.to_goom(Jr)
    Lo = L or 128  # the library's default
    say(f"reset always T={T} d={d} L={L or 'default'} {np.dtype(ctype).name}")
    states, flags, growth = G.scan_reset(dev(Jz), chunk_len=L, policy=RESET_ALWAYS)
    re, sg, oflag, ogrowth = oracle.reset_scan(Jz, None, check_every=Lo, policy=1)
    assert np.array_equal(host(flags), oflag)
    # Chunk products, carries and the factorisations at the resets run in double on the GPU, as in the oracle,
    # so every entry of every state is compared, whatever the chunk length, with one exception: the orthonormal
    # factor of a reset is good to about cond^2 2^-53 of a column's NORM (1e-9 at a condition number of 3000; with
    # double components a second factorisation brings that to rounding level), so entries below e^-10 (e^-9) of
    # their column's largest are left out; the log prints their share.
    got = host(states)
    tiny = re < re.max(axis=1, keepdims=True) - (10.0 if comp == np.float32 else 9.0)
    well = ~tiny
    if comp == np.float64:
        # at 1e-10 the orthonormal factor's own conditioning shows (a perturbation of the state by one part in
        # 2^53 moves the factor by cond times as much): the oracle's finite-difference probe masks such entries
        def fn(mats):
            r, s_, _, _ = oracle.reset_scan(mats, None, check_every=Lo, policy=1)
            return r, s_, np.ones_like(r)
        _, _, _, wellfd = with_sensitivity(fn, [Jz], comp, nprobe=2)
        well &= wellfd
    compare(got, re, sg, None, name=f"reset always T{T}d{d}L{Lo}", max_ill_fraction=0.1 if comp == np.float32 else 0.3, well=well)
    vg = np.where(got.imag != 0, -1.0, 1.0) * np.exp(got.real.astype(np.float64) - re.max(axis=1, keepdims=True))
    vr = np.where(sg == 1, -1.0, 1.0) * np.exp(re - re.max(axis=1, keepdims=True))
    col_err = np.linalg.norm(vg - vr, axis=1) / np.linalg.norm(vr, axis=1)
    say(f"  column-wise relative error of the states: max {col_err.max():.2e}")
    assert col_err.max() < (1e-6 if comp == np.float32 else 1e-9)
    lam_gpu = host(growth) / (T * 0.01)
    lam_ref = ogrowth / (T * 0.01)
    lam_qr = oracle.lyapunov_qr(Jr.astype(np.float64), 0.01)
    say(f"  exponents: max |gpu - reset oracle| = {np.abs(lam_gpu - lam_ref).max():.2e}, max |gpu - QR oracle| = {np.abs(lam_gpu - lam_qr).max():.2e}")
    assert np.abs(lam_gpu - lam_ref).max() < 1e-9 and np.abs(lam_gpu - lam_qr).max() < 1e-4


@pytest.mark.parametrize("T,d,batch,ctype,policy,thr", [(11, 4, 2, np.complex128, 0, 0.9), (37, 8, 1, np.complex128, 0, 0.97), (64, 16, 1, np.complex128, 0, 0.9),
                                                        (23, 6, 2, np.complex64, 0, 0.9), (40, 32, 1, np.complex64, 0, 0.8), (9, 4, 1, np.complex64, -1, 0.9),
                                                        (9, 4, 1, np.complex128, 1, 0.9), (33, 64, 1, np.complex128, 0, 0.7), (12, 96, 1, np.complex128, 0, 0.5),
                                                        (6, 128, 1, np.complex64, 1, 0.9)])
def test_reset_scan_in_the_papers_tree_order(G, oracle, T, d, batch, ctype, policy, thr):
    """The selective-resetting transformation applied in the order of the paper's own parallel scan (Section 5, eq. 28;
    Appendix C) against the oracle's literal (A*, B*) tuples over reals in the same order.  Which compounds are reset is
    decided by cosines; the inputs are drawn so that no decision sits near its threshold (checked on the oracle side)."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(100 + T + d)
    A = (rng.standard_normal((batch, T, d, d)) / math.sqrt(d) * 1.5).astype(comp)
    X0 = rng.standard_normal((batch, d, d)).astype(comp)
    say(f"tree-order reset scan T={T} d={d} batch={batch} {np.dtype(ctype).name} policy={policy} threshold={thr}")
    states, flags = G.scan_reset_tree(dev(oracle.to_goom(A)), dev(oracle.to_goom(X0)), policy=policy, cos_threshold=thr)
    got, gflags = host(states), host(flags)
    nreset = 0
    for b in range(batch):
        want, was = oracle.reset_scan_tree_real(X0[b].astype(np.float64), A[b].astype(np.float64), policy=policy, cos_threshold=thr)
        # decisions are robust: the same flags come out with the threshold moved a little either way
        for dthr in (-1e-3, 1e-3):
            if policy == 0:
                assert np.array_equal(oracle.reset_scan_tree_real(X0[b].astype(np.float64), A[b].astype(np.float64), policy=policy, cos_threshold=thr + dthr)[1], was)
        assert np.array_equal(gflags[b].astype(bool), was[1:])
        nreset += int(was[1:].sum())
        val = np.where(got[b].imag != 0, -1.0, 1.0) * np.exp(got[b].real.astype(np.float64))
        err = np.linalg.norm(val - want[1:], axis=1) / np.linalg.norm(want[1:], axis=1)
        # The float path forms every compound with float products, and an orthonormal factor's later columns hang on
        # the small differences between nearly parallel columns: columns that move by more than 1/16 of the bound
        # when the oracle's inputs are perturbed by 64 units in the last place of the component type (a compound of
        # 2^k elements has been through k float products of d terms each, about k sqrt(d) units relative to a column's
        # norm) are left out
        bound = 2e-4 if comp == np.float32 else 1e-9
        eta = 2.0 ** -18 if comp == np.float32 else 2.0 ** -47
        sens = np.zeros((T, d))
        for _ in range(4):  # (the last column of a factor can flip its sign outright: several probes, so that one of them shows it)
            pert, pwas = oracle.reset_scan_tree_real(X0[b].astype(np.float64) * (1 + eta * rng.standard_normal((d, d))),
                                                     A[b].astype(np.float64) * (1 + eta * rng.standard_normal((T, d, d))), policy=policy, cos_threshold=thr)
            assert np.array_equal(pwas, was)
            sens = np.maximum(sens, np.linalg.norm(pert[1:] - want[1:], axis=1) / np.linalg.norm(want[1:], axis=1))
        well = sens <= bound / 16
        say(f"  item {b}: {int(was[1:].sum())} of {T} states descend from a reset; column-wise relative error max {err[well].max():.2e} "
            f"over the {well.mean():.1%} of the columns that are determined at this precision")
        assert err[well].max() < bound and well.mean() > (0.1 if comp == np.float32 else 0.9)
    if policy == 0:
        assert nreset > 0
    # S == 0: the plain scan
    if policy == -1:
        plain = host(G.scan(dev(oracle.to_goom(A)), init=dev(oracle.to_goom(X0))))
        assert np.allclose(plain.real, got.real, rtol=1e-4, atol=1e-3) and np.array_equal(plain.imag != 0, got.imag != 0)


@pytest.mark.parametrize("T,d,L,thr", [(400, 8, 10, 0.9), (90, 80, 3, 0.6)])
def test_reset_scan_colinear_policy_and_initial_state(G, oracle, T, d, L, thr):
    from paper_2510_03426_amd import RESET_COLINEAR
    # (d = 80: products of N(0,1) matrices, whose columns turn colinear within a few steps; the near-identity
    # Jacobians that stand in for Lorenz-96 above d = 40 never do)
    Jr = lorenz_chain(T, d, 62) if d <= 40 else si.normal_chain(si.BASE_SEED + 62, T, d)
    Jz = oracle.to_goom(Jr)
    S0 = oracle.to_goom(si.normal_init(si.BASE_SEED + 62, d, d))
    states, flags, growth = G.scan_reset(dev(Jz), dev(S0), chunk_len=L, policy=RESET_COLINEAR, cos_threshold=thr)
    re, sg, oflag, ogrowth = oracle.reset_scan(Jz, S0, check_every=L, policy=0, cos_threshold=thr)
    gflag = host(flags)
    say(f"  colinear policy: {int(gflag.sum())} resets on the GPU, {int(oflag.sum())} in the oracle")
    assert 0 < oflag.sum() < T // L
    assert np.array_equal(gflag, oflag)
    assert np.abs(host(growth) - ogrowth).max() < 1e-3 * T * 0.01


def test_lyapunov_spectrum_lorenz96(G, oracle):
    # Lorenz-96, d = 32: spectrum from the reset scan against step-by-step QR in double
    T, d = 16384, 32
    Jr = lorenz_chain(T, d, 4, burn_in=10000)
    lam_qr = oracle.lyapunov_qr(Jr, 0.01)
    Jz = dev(oracle.to_goom(Jr))
    # The spectrum has a nearly degenerate pair (exponents 25 and 26): how growth is split between
    # the two is the least determined quantity here, and the float chunk products show it first.
    # Chunks of up to 32 steps (the default) keep every exponent within 1e-3; longer chunks trade
    # accuracy of that pair for a shorter serial phase, with the pair's sum still accurate.
    for L, bound in ((0, 1e-3), (16, 1e-3), (32, 1e-3), (64, 5e-3)):
        lam = host(G.lyapunov_spectrum(Jz, 0.01, chunk_len=L))
        err = np.abs(lam - lam_qr)
        both = abs((lam[24] + lam[25]) - (lam_qr[24] + lam_qr[25]))
        say(f"  L={L or 'default'}: max |lambda_gpu - lambda_qr| = {err.max():.2e} at k={int(err.argmax()) + 1} "
            f"(sum of exponents 25 and 26 off by {both:.2e}); lambda_1 = {lam[0]:.4f}, sum = {lam.sum():.3f}")
        assert err.max() < bound and both < 1e-3 and abs(lam.sum() - lam_qr.sum()) < 1e-3
    want_sum = np.mean([np.linalg.slogdet(j.astype(np.float64))[1] for j in Jr[::16]]) / 0.01
    assert abs(lam.sum() - want_sum) < 0.5


def test_lyapunov_spectrum_gaussian_closed_form(G, oracle):
    # products of i.i.d. N(0,1) matrices: lambda_k = (ln 2 + psi((d - k + 1) / 2)) / 2
    from scipy.special import digamma
    T, d = 20000, 16
    x = si.normal_chain(si.BASE_SEED + 63, T, d)
    # the exponents spread over 2 nats per step here, so a chunk may only span a few steps before
    # the most contracted direction drops below float resolution (e^-16 after 8 steps)
    lam = host(G.lyapunov_spectrum(dev(oracle.to_goom(x)), 1.0, chunk_len=3))
    want = 0.5 * (math.log(2) + digamma((d - np.arange(1, d + 1) + 1) / 2))
    say(f"  gaussian spectrum: max deviation from closed form {np.abs(lam - want).max():.3f}")
    assert np.abs(lam - want).max() < 0.06
    lam_qr = oracle.lyapunov_qr(x.astype(np.float64), 1.0)
    assert np.abs(lam - lam_qr).max() < 1e-3


# ------------------------------------ per-step estimator and largest exponent (Sections 4.2.1-4.2.2)

@pytest.mark.parametrize("T,d,L,policy,ctype", [(2048, 32, 0, 1, np.complex64), (1000, 8, 16, 1, np.complex64), (600, 16, 7, 0, np.complex64),
                                                (300, 64, 16, 1, np.complex64), (1500, 32, 0, 1, np.complex128), (400, 10, 9, 0, np.complex128),
                                                (200, 64, 16, 1, np.complex128), (96, 100, 12, 1, np.complex64), (64, 128, 16, 1, np.complex128)])
def test_lyapunov_per_step_estimator(G, oracle, T, d, L, policy, ctype):
    # groups (b)-(d): two QRs per step on the selectively reset states; against the same groups in the
    # oracle (fed the oracle's own states) and against the sequential QR method
    dt = 0.01
    Jr = lorenz_chain(T, d, 71, burn_in=3000)
    if ctype == np.complex128:
        Jr = Jr.astype(np.float64)
    Jz = oracle.to_goom(Jr)
    assert Jz.dtype == ctype
    check = L if L > 0 else 32
    re, sg, _, _ = oracle.reset_scan(Jz, None, check_every=check, policy=policy)
    eye_re = np.where(np.eye(d) > 0, 0.0, -np.inf)
    prev = (np.concatenate([eye_re[None], re[:-1]]), np.concatenate([np.zeros((1, d, d), np.uint8), sg[:-1]]))
    lam_ref, logs_ref = oracle.lyapunov_from_states(prev, Jr, dt)
    lam_qr = oracle.lyapunov_qr(Jr, dt)
    lam, logs = G.lyapunov_spectrum_per_step(dev(Jz), dt, chunk_len=L, policy=policy, want_step_logs=True)
    lam, logs = host(lam), host(logs)
    say(f"per-step estimator {np.dtype(ctype).name} T={T} d={d} L={L or 'default'} policy={policy}: max |gpu - oracle groups| = "
        f"{np.abs(lam - lam_ref).max():.2e}, max |gpu - QR method| = {np.abs(lam - lam_qr).max():.2e}, "
        f"worst single log R_kk off by {np.abs(logs - logs_ref).max():.2e}")
    tol = 1e-3 if ctype == np.complex64 else 1e-7
    assert np.abs(lam - lam_ref).max() < tol and np.abs(lam - lam_qr).max() < 1e-3
    # per step the logs add up to log|det J_t| whatever the basis; float QR keeps that to about 1e-4
    dets = np.array([np.linalg.slogdet(j.astype(np.float64))[1] for j in Jr])
    assert np.abs(logs.sum(axis=1) - dets).max() < (2e-3 if ctype == np.complex64 else 1e-9)
    # and the estimator that accumulates growth at the resets agrees
    lam2 = host(G.lyapunov_spectrum(dev(Jz), dt, chunk_len=L, policy=1))
    assert np.abs(lam - lam2).max() < 1e-3


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_largest_lyapunov_exponent(G, oracle, ctype):
    comp = np.float32 if ctype == np.complex64 else np.float64
    dt = 0.01
    for T, d, batch in ((4096, 32, 2), (700, 8, 3)):
        Js, us, want, std = [], [], [], []
        for b in range(batch):
            Jr = lorenz_chain(T, d, 80 + b, burn_in=3000)
            u0 = si.normal_f32(si.BASE_SEED + 90 + b, 4, d).astype(np.float64)
            u0 /= np.linalg.norm(u0)
            Jz, uz = oracle.to_goom(Jr.astype(comp)), oracle.to_goom(u0.astype(comp))
            Js.append(Jz)
            us.append(uz)
            want.append(oracle.lle_goom(Jz, uz, dt, scaled=True))
            std.append(oracle.lle_standard(Jr, u0, dt))
        got = host(G.largest_lyapunov(dev(np.stack(Js)), dt, u0=dev(np.stack(us))))
        say(f"LLE {np.dtype(ctype).name} T={T} d={d}: gpu {got}, oracle (eq. 24) {np.array(want)}, normalised iteration {np.array(std)}")
        assert np.abs(got - np.array(want)).max() < 1e-3 and np.abs(got - np.array(std)).max() < 1e-3
        # default start vector: all entries 1 / sqrt(d)
        got0 = host(G.largest_lyapunov(dev(np.stack(Js)), dt))
        u = np.full(d, 1.0 / math.sqrt(d))
        ref0 = np.array([oracle.lle_standard(lorenz_chain(T, d, 80 + b, burn_in=3000), u, dt) for b in range(batch)])
        assert np.abs(got0 - ref0).max() < 1e-3
    # Gaussian factors far past float range: closed form (ln 2 + psi(d / 2)) / 2
    from scipy.special import digamma
    T, d = 20000, 16
    Gz = oracle.to_goom(si.normal_chain(si.BASE_SEED + 95, T, d).astype(comp))
    got = float(host(G.largest_lyapunov(dev(Gz), 1.0)))
    lam = 0.5 * (math.log(2.0) + digamma(d / 2))
    say(f"  Gaussian d={d}: {got:.5f} (closed form {lam:.5f}), log-norm {got * T:.0f}")
    assert abs(got - lam) < 0.01 and got * T > 2.0e4


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_scaled_exponentiation(G, oracle, ctype):
    # the scaled exponentiation (Section 4.3, eq. 27) on states of a recurrence whose magnitudes leave float range, and on ragged shapes
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(77)
    for shape in ((3, 1000, 32), (513, 5), (70, 100), (2, 64), (9, 1)):
        re = rng.normal(0.0, 400.0, shape)
        z = (re + 1j * np.pi * rng.integers(0, 2, shape)).astype(ctype)
        z.imag[...] = np.where(z.imag != 0, comp(np.pi), comp(0))
        if shape[-1] > 2:
            z.real[0, ..., 1] = -np.inf  # a zero entry
        want, cw = oracle.scaled_exp(z)
        got, c = G.scaled_exp(dev(z), want_logscale=True)
        got, c = host(got), host(c)
        assert np.array_equal(c, cw.astype(comp))
        eps = np.finfo(comp).eps
        # the argument re - c + 2 is formed in double on the device: its rounding, |argument| 2^-53,
        # is the relative error of the exponential (visible only with double components)
        arg = np.abs(np.where(np.isfinite(z.real), z.real - cw[..., None], 0.0))
        assert np.all(np.abs(got - want) <= (4 * eps + 2.0 ** -52 * arg) * np.abs(want) + np.finfo(comp).tiny), np.abs(got - want).max()
        assert np.abs(got).max() <= math.e ** 2 * (1 + 4 * eps)
    zero = dev(np.full((4, 8), -np.inf + 0j).astype(ctype))
    got, c = G.scaled_exp(zero, want_logscale=True)
    assert np.all(host(got) == 0) and np.all(np.isneginf(host(c)))
    # end to end: states of the recurrence, scaled
    A, b = si.recurrence_inputs(si.BASE_SEED + 55, 2, 4000, 16, gain=1.3)
    Az, bz = oracle.to_goom(A.astype(comp)), oracle.to_goom(b.astype(comp))
    H = G.affine_scan(dev(Az), dev(bz))
    want, _ = oracle.scaled_exp(host(H))
    got = host(G.scaled_exp(H))
    assert host(H).real.max() > 700 and np.all(np.abs(got - want) <= 4 * eps * np.abs(want) + np.finfo(comp).tiny)


@pytest.mark.parametrize("T,d,batch,chunk,ctype,ti,gain", [
    (300, 32, 3, 32, np.complex64, False, 1.05),   # scaled states written by the walk itself
    (1000, 16, 2, 7, np.complex64, False, 1.05),
    (4000, 16, 2, 0, np.complex64, False, 1.3),    # magnitudes far outside float range
    (500, 32, 2, 25, np.complex64, True, 1.0),     # constant matrix
    (400, 64, 2, 20, np.complex64, True, 1.0),     # constant 64 x 64 matrix: scaled states by the walk
    (64, 8, 2, 0, np.complex64, False, 1.05),      # scaled states by the vector chains, a single chunk
    (257, 64, 1, 40, np.complex64, False, 1.05),
    (200, 16, 2, 16, np.complex128, False, 1.05),
    (40, 32, 2, 0, np.complex64, False, 1.05),     # a single chunk
    (121, 32, 122, 0, np.complex64, False, 1.05),   # many sequences: scaled states written by the sequential walk
    (3000, 32, 120, 0, np.complex64, False, 1.3),   # the same, magnitudes far outside float range
])
def test_affine_scan_scaled_states(G, oracle, T, d, batch, chunk, ctype, ti, gain):
    # the scaled exponentiation (Section 4.3, eq. 27) applied to the recurrence's states inside the scan: against the oracle's states, scaled by
    # the oracle.  An entry is compared where it and its vector's largest entry are well conditioned.
    comp = np.float32 if ctype == np.complex64 else np.float64
    A, b = si.recurrence_inputs(si.BASE_SEED + 57, batch, T, d, gain=gain)
    if ti:
        A = A[:, :1] * np.float32(0.9)
    Az, bz = oracle.to_goom(A.astype(comp)), oracle.to_goom(b.astype(comp))
    say(f"affine scaled T={T} d={d} batch={batch} chunk={chunk} {ctype.__name__} ti={ti}")
    fn = lambda a_, b_: oracle.affine_scan(np.ascontiguousarray(np.broadcast_to(a_, (batch, T, d, d))), b_, h0=None, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [Az, bz], comp)
    want, cw = oracle.scaled_exp(re + 1j * np.pi * sg)
    got, c = G.affine_scan_scaled(dev(Az[:, 0] if ti else Az), dev(bz), chunk_len=chunk, time_invariant=ti, want_logscale=True)
    got, c = host(got).astype(np.float64), host(c).astype(np.float64)
    assert got.shape == (batch, T, d) and c.shape == (batch, T)
    top = np.argmax(np.where(np.isfinite(re), re, -np.inf), axis=-1)
    top_well = np.take_along_axis(well, top[..., None], axis=-1)[..., 0]
    ok = well & top_well[..., None]
    assert ok.mean() > 0.8, ok.mean()
    # the bar for log-magnitudes carried over: d(ln scaled_i) = d(re_i) - d(c), each within its tolerance
    def bound(re_, cw_):
        with np.errstate(invalid="ignore"):
            return np.where(np.isfinite(re_), tolerance(re_, comp), 0.0) + tolerance(cw_, comp)[..., None]
    ratio = (np.abs(got - want) / (bound(re, cw) * np.abs(want) + 1e-30))[ok]
    say(f"  worst error / bound {ratio.max():.3g}")
    assert ratio.max() <= 1
    assert np.all(np.abs(got) <= math.e ** 2 * (1 + 1e-5))
    assert np.all(np.abs(c - cw)[top_well] <= tolerance(cw, comp)[top_well])
    if gain > 1.2:
        assert cw.max() > 700
    # without the log scales, and with an initial state
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 58, 9, batch * d).reshape(batch, d).astype(comp))
    fn0 = lambda a_, b_, h_: oracle.affine_scan(np.ascontiguousarray(np.broadcast_to(a_, (batch, T, d, d))), b_, h0=h_, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn0, [Az, bz, h0], comp)
    want, cw = oracle.scaled_exp(re + 1j * np.pi * sg)
    got = host(G.affine_scan_scaled(dev(Az[:, 0] if ti else Az), dev(bz), dev(h0), chunk_len=chunk, time_invariant=ti)).astype(np.float64)
    top = np.argmax(np.where(np.isfinite(re), re, -np.inf), axis=-1)
    ok = well & np.take_along_axis(well, top[..., None], axis=-1)
    ratio = (np.abs(got - want) / (bound(re, cw) * np.abs(want) + 1e-30))[ok]
    assert ratio.max() <= 1


# ------------------------------------------------------------------ backward passes (Sections 3.1, 4.3)

@pytest.mark.parametrize("comp", [np.float32, np.float64])
def test_codec_backward_redefined_derivatives(G, oracle, comp):
    rng = np.random.default_rng(90)
    n = (1 << 16) + 7
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-30, 30, n))).astype(comp)
    x[:8] = [0.0, -0.0, 1.0, -1.0, 1e-30, -1e-30, 3.0, -3.0]
    g = rng.standard_normal(n).astype(comp)
    eps = float(np.finfo(comp).eps)
    got = host(G.to_goom_backward(dev(x), dev(g), eps)).astype(np.float64)
    want = oracle.to_goom_backward(x, g, eps)
    assert np.all(np.abs(got - want) <= 2 * np.finfo(comp).eps * np.abs(want)) and np.all(np.isfinite(got)) and np.all(got[g != 0] != 0)
    z = oracle.to_goom(x)
    got = host(G.from_goom_backward(dev(z), dev(g), eps)).astype(np.float64)
    want = oracle.from_goom_backward(z, g, eps)
    assert np.all(np.abs(got - want) <= 4 * np.finfo(comp).eps * np.abs(want) + np.finfo(comp).tiny) and np.all(got[g != 0] != 0)


@pytest.mark.parametrize("T,d,batch,chunk,ctype,with_h0,gain", [
    (300, 32, 2, 32, np.complex64, False, 1.05), (1000, 16, 2, 0, np.complex64, True, 1.05), (4000, 32, 1, 0, np.complex64, True, 1.3),
    (64, 8, 3, 9, np.complex64, True, 1.05), (257, 64, 1, 40, np.complex64, False, 1.05), (200, 16, 2, 16, np.complex128, True, 1.05),
    (1, 32, 2, 0, np.complex64, True, 1.05), (40, 128, 1, 8, np.complex128, True, 1.05), (50, 31, 2, 0, np.complex64, False, 1.05),
    (601, 16, 2, 50, np.complex64, False, 1.05),
    # many sequences of d = 32: the adjoint recurrence walked sequence by sequence, its factors read transposed and in reverse
    (300, 32, 96, 0, np.complex64, False, 1.05), (37, 32, 100, 0, np.complex64, True, 1.05), (1, 32, 96, 0, np.complex64, True, 1.05)])
def test_affine_scan_backward(G, oracle, T, d, batch, chunk, ctype, with_h0, gain):
    """Gradients of L = sum grad_h * Re h with respect to the log-magnitudes of A, bias and h0, against the oracle's
    adjoint recurrence fed the same forward states."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    A, b = si.recurrence_inputs(si.BASE_SEED + 91, batch, T, d, gain=gain)
    Az, bz = oracle.to_goom(A.astype(comp)), oracle.to_goom(b.astype(comp))
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 92, 9, batch * d).reshape(batch, d).astype(comp)) if with_h0 else None
    Gh = si.normal_f32(si.BASE_SEED + 93, 10, batch * T * d).reshape(batch, T, d).astype(comp)
    say(f"affine backward T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name} h0={with_h0}")
    Hd = G.affine_scan(dev(Az), dev(bz), None if h0 is None else dev(h0), chunk_len=chunk)
    H = host(Hd)
    ga, gb, gh0 = G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), None if h0 is None else dev(h0), chunk_len=chunk)
    ga, gb = host(ga).astype(np.float64), host(gb).astype(np.float64)
    wa, wb, wh0, (lre, lsg) = oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)
    if gain > 1.2:
        assert H.real.max() > 700 and lre.min() < -700  # states and adjoints far outside float range, gradients not
    # conditioning, decided by the oracle alone: the adjoints are signed sums; where half-unit perturbations of the
    # inputs' log-magnitudes move a gradient by more than 1/16 of the tolerance the entry is left out
    rng = np.random.default_rng(5)
    eta = 2.0 ** -24 if comp == np.float32 else 2.0 ** -53
    rel = 1e-3 if comp == np.float32 else 1e-9
    tol_a = rel * np.abs(wa) + 1e-3 * rel * np.abs(wa).max(axis=(-1, -2), keepdims=True) + 2 * float(np.finfo(comp).tiny)  # (results are reals of the component type; subnormal ones may be flushed)
    tol_b = rel * np.abs(wb) + 1e-3 * rel * np.abs(wb).max(axis=-1, keepdims=True) + 2 * float(np.finfo(comp).tiny)
    sens_a, sens_b = np.zeros_like(wa), np.zeros_like(wb)
    for _ in range(4 if wa.size > 500000 * d else 2):  # (more probes where there are many more entries: see test_affine_scan_matches_oracle)
        pert = lambda z: None if z is None else (z.astype(np.complex128) + eta * rng.standard_normal(z.shape) * np.where(np.isfinite(z.real), 1.0, 0.0))
        pa, pb, _, _ = oracle.affine_scan_backward(pert(Az), pert(bz), Gh, h0=pert(h0), h=pert(H))
        sens_a, sens_b = np.maximum(sens_a, np.abs(pa - wa)), np.maximum(sens_b, np.abs(pb - wb))
    well_a, well_b = sens_a <= tol_a / 16, sens_b <= tol_b / 16
    ra = (np.abs(ga - wa) / tol_a)[well_a].max()
    rb = (np.abs(gb - wb) / tol_b)[well_b].max()
    say(f"  worst error / tolerance: grad A {ra:.3g}, grad bias {rb:.3g}; left out as ill conditioned {1 - well_a.mean():.2e} / {1 - well_b.mean():.2e}")
    # (an expansive recurrence makes a quarter of its adjoints cancelling sums; the logs print the share)
    min_well = 0.7 if gain > 1.2 else 0.9
    assert ra <= 1 and rb <= 1 and well_a.mean() > min_well and well_b.mean() > min_well
    sig = well_a & (np.abs(wa) > 2 * tol_a)  # signs wherever the tolerance does not reach zero
    assert np.array_equal(np.signbit(ga)[sig], np.signbit(wa)[sig])
    if with_h0:
        gh0 = host(gh0).astype(np.float64)
        assert np.all(np.abs(gh0 - wh0) <= 2e-3 * np.abs(wh0) + 1e-4 * np.abs(wh0).max())
    else:
        assert np.all(ga[:, 0] == 0)  # the first matrix multiplies a zero vector


@pytest.mark.parametrize("shape,ctype,flags,spread", [
    ((3, 16, 16, 16), np.complex64, 0, 0.0), ((2, 37, 50, 29), np.complex64, 0, 4000.0), ((2, 128, 128, 128), np.complex64, 0, 300.0),
    ((2, 128, 128, 128), np.complex64, 1, 4000.0), ((1, 200, 130, 70), np.complex64, 0, 4000.0), ((5, 8, 64, 1), np.complex64, 0, 100.0),
    ((2, 1, 1, 1), np.complex64, 0, 50.0), ((2, 40, 24, 56), np.complex128, 0, 4000.0), ((1, 128, 128, 128), np.complex128, 0, 1e5),
    ((2, 64, 32, 100), np.complex64, 1, 1000.0), ((1, 70, 150, 40), np.complex128, 0, 500.0)])
def test_lmme_backward(G, oracle, shape, ctype, flags, spread):
    """Gradients of a loss with respect to the log-magnitudes of both operands of an LMME, against the oracle fed the
    same forward result.  Every gradient is a signed sum of terms G_ik A_ij B_jk / C_ik; the bound is on the error
    relative to the sum of their magnitudes (the oracle's own sums on operands with all signs positive), which is what
    a product in the component type can hold."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    b, n, d, m = shape
    rng = np.random.default_rng(17)
    say(f"lmme backward batch={b} n={n} d={d} m={m} {np.dtype(ctype).name} flags={flags} spread={spread}")
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 95, 7, b * n * d).reshape(b, n, d).astype(comp))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 96, 8, b * d * m).reshape(b, d, m).astype(comp))
    A.real += rng.uniform(-spread, spread, (b, n, 1)).astype(comp)  # rows and columns far outside float range
    B.real += rng.uniform(-spread, spread, (b, 1, m)).astype(comp)
    Gc = si.normal_f32(si.BASE_SEED + 97, 10, b * n * m).reshape(b, n, m).astype(comp)
    if n * d > 8:
        A[0, 0, 1] = -np.inf      # a zero entry
        Gc[0, n - 1, 0] = 0.0     # an output the loss does not see
    Cd = G.lmme(dev(A), dev(B), flags=flags)
    Cz = host(Cd)
    if n > 2 and m > 2:
        Cz[b - 1, 1, 2] = -np.inf  # an output taken to be exactly zero passes no gradient
        Cd = dev(Cz)
    ga, gb = G.lmme_backward(dev(A), dev(B), Cd, dev(Gc), flags=flags)
    ga, gb = host(ga).astype(np.float64), host(gb).astype(np.float64)
    wa, wb = oracle.lmme_backward(A, B, Gc, c=Cz)
    ma, mb = oracle.lmme_backward(A.real + 0j, B.real + 0j, np.abs(Gc), c=Cz.real + 0j)  # sums of the terms' magnitudes
    assert np.all(ma >= np.abs(wa) * (1 - 1e-12)) and np.all(mb >= np.abs(wb) * (1 - 1e-12))
    rel = 1e-5 if comp == np.float32 else 1e-11
    tiny = 2 * float(np.finfo(comp).tiny)  # (results are reals of the component type; subnormal ones may be flushed)
    ea, eb = np.abs(ga - wa) / (rel * ma + tiny), np.abs(gb - wb) / (rel * mb + tiny)
    say(f"  worst error / tolerance: grad A {ea.max():.3g}, grad B {eb.max():.3g}; largest |grad| {np.abs(wa).max():.3g}")
    assert np.isfinite(ga).all() and np.isfinite(gb).all()
    assert ea.max() <= 1 and eb.max() <= 1
    sig_a, sig_b = np.abs(wa) > 2 * (rel * ma + tiny), np.abs(wb) > 2 * (rel * mb + tiny)
    assert np.array_equal(np.signbit(ga)[sig_a], np.signbit(wa)[sig_a]) and np.array_equal(np.signbit(gb)[sig_b], np.signbit(wb)[sig_b])
    if n * d > 8:
        assert ga[0, 0, 1] == 0.0
    # the sum rules, on the device results alone: the gradients of row i of A' add up to those of row i of C' that pass
    live = np.where(np.isneginf(Cz.real), 0.0, Gc.astype(np.float64))
    assert np.all(np.abs(ga.sum(axis=2) - live.sum(axis=2)) <= 4 * rel * ma.sum(axis=2) + 1e-30)
    assert np.all(np.abs(gb.sum(axis=1) - live.sum(axis=1)) <= 4 * rel * mb.sum(axis=1) + 1e-30)


@pytest.mark.parametrize("T,d,m,batch,chunk,ctype,with_init", [
    (40, 8, 8, 2, 0, np.complex64, False), (300, 16, 16, 2, 16, np.complex64, True), (257, 32, 8, 1, 0, np.complex64, True),
    (60, 64, 64, 1, 0, np.complex64, False), (60, 24, 40, 2, 7, np.complex128, True), (1, 16, 16, 2, 0, np.complex64, True),
    (30, 100, 60, 1, 0, np.complex64, True), (2000, 16, 16, 1, 0, np.complex64, False), (1, 8, 8, 1, 0, np.complex128, False),
    (500, 12, 5, 3, 50, np.complex64, True), (12, 200, 100, 1, 0, np.complex64, True), (10, 136, 136, 1, 4, np.complex128, False)])
def test_scan_backward(G, oracle, T, d, m, batch, chunk, ctype, with_init):
    """Gradients of L = sum grad_p * Re p with respect to the log-magnitudes of every factor and of the initial state,
    against the oracle's adjoint recurrence fed the same forward states."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    Z = oracle.to_goom(si.normal_f32(si.BASE_SEED + 101, 1, batch * T * d * d).reshape(batch, T, d, d).astype(comp))
    S0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 102, 2, batch * d * m).reshape(batch, d, m).astype(comp)) if with_init else None
    Gp = si.normal_f32(si.BASE_SEED + 103, 10, batch * T * d * m).reshape(batch, T, d, m).astype(comp)
    if T > 3:
        Z[0, 2, 1, 0] = -np.inf   # a zero entry of a factor
        Gp[0, 1, 0, 0] = 0.0      # an entry the loss does not see
    say(f"scan backward T={T} d={d} m={m} batch={batch} chunk={chunk} {np.dtype(ctype).name} init={with_init}")
    Pd = G.scan(dev(Z), None if S0 is None else dev(S0), chunk_len=chunk)
    P = host(Pd)
    gm, gi = G.scan_backward(dev(Z), Pd, dev(Gp), None if S0 is None else dev(S0), chunk_len=chunk)
    gm = host(gm).astype(np.float64)
    gi = None if gi is None else host(gi).astype(np.float64)
    assert np.isfinite(gm).all()
    if T >= 2000:
        assert P.real.max() > 2000  # states far outside float range, gradients not
    rng = np.random.default_rng(6)
    eta = 2.0 ** -24 if comp == np.float32 else 2.0 ** -53
    rel = 1e-3 if comp == np.float32 else 1e-9
    tiny = 2 * float(np.finfo(comp).tiny)
    worst, worst_well, kept = 0.0, 0.0, []
    for b in range(batch):
        s0 = None if S0 is None else S0[b]
        wm, wi, _ = oracle.scan_backward(Z[b], Gp[b], init=s0, p=P[b])
        # conditioning, decided by the oracle alone: the adjoints are signed sums.  The probe moves every input's log-magnitude by
        # a half unit in the last place, independently, and records how far each gradient moves.  The kernels round every one
        # of the T sums of d + m products an adjoint passes through, a random walk of sqrt(T (d + m)) such half units: every
        # entry has to lie within the tolerance plus that many times what the probes moved it.
        tol = rel * np.abs(wm) + 1e-3 * rel * np.abs(wm).max(axis=(-1, -2), keepdims=True) + tiny
        sens = np.zeros_like(wm)
        pert = lambda z: None if z is None else (z.astype(np.complex128) + eta * rng.standard_normal(z.shape) * np.where(np.isfinite(z.real), 1.0, 0.0))
        for _ in range(2):
            pm, _, _ = oracle.scan_backward(pert(Z[b]), Gp[b], init=pert(s0), p=pert(P[b]))
            sens = np.maximum(sens, np.abs(pm - wm))
        noise = math.sqrt(T * (d + m)) * sens
        worst = max(worst, (np.abs(gm[b] - wm) / (tol + noise)).max())
        well = noise <= tol
        kept.append(well.mean())
        worst_well = max(worst_well, (np.abs(gm[b] - wm) / tol)[well].max())
        sig = np.abs(wm) > 2 * (tol + noise)
        assert np.array_equal(np.signbit(gm[b])[sig], np.signbit(wm)[sig])
        if with_init:
            assert np.all(np.abs(gi[b] - wi) <= 2 * rel * np.abs(wi) + 1e-2 * rel * np.abs(wi).max() + tiny)
        if T > 3 and b == 0:
            assert gm[0, 2, 1, 0] == 0.0
    say(f"  worst error / bound of grad M {worst:.3g}; entries whose bound is the tolerance alone (within a factor 2): {min(kept):.3f}, "
        f"their worst error / tolerance {worst_well:.3g}")
    assert worst <= 1 and min(kept) > (0.1 if comp == np.float32 else 0.99)  # (the share only shows that the bound is not all noise)
    # the sum rule on the device results alone: the gradients of the last factor's row i add up to those of row i of the last state
    assert np.all(np.abs(gm[:, -1].sum(axis=2) - Gp[:, -1].astype(np.float64).sum(axis=2)) <= 50 * rel * np.abs(gm[:, -1]).sum(axis=2) + 1e-30)


@pytest.mark.parametrize("T,d,batch,chunk,ctype,with_h0,gain", [
    (3000, 32, 2, 0, np.complex64, True, 1.02), (1000, 16, 3, 0, np.complex64, False, 1.02), (300, 8, 2, 16, np.complex64, True, 1.02),
    (200, 64, 1, 40, np.complex64, True, 0.95), (150, 16, 2, 16, np.complex128, True, 1.02), (40, 100, 1, 8, np.complex128, False, 1.0),
    (1, 32, 2, 0, np.complex64, True, 1.02), (700, 32, 1, 7, np.complex64, False, 1.1)])
def test_affine_scan_backward_time_invariant(G, oracle, T, d, batch, chunk, ctype, with_h0, gain):
    """The recurrence with one matrix for all steps (the paper's state-space layer): the matrix's gradient is the sum over
    the steps of lam_t[i] A[i, j] h_{t-1}[j]; bias and initial-state gradients as in the time-varying pass."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    A, _ = si.recurrence_inputs(si.BASE_SEED + 111, batch, 1, d, gain=gain)
    _, b = si.recurrence_inputs(si.BASE_SEED + 112, batch, T, d)
    Az, bz = oracle.to_goom(A[:, 0].astype(comp)), oracle.to_goom(b.astype(comp))
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 113, 9, batch * d).reshape(batch, d).astype(comp)) if with_h0 else None
    Gh = si.normal_f32(si.BASE_SEED + 114, 10, batch * T * d).reshape(batch, T, d).astype(comp)
    say(f"time-invariant affine backward T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name} h0={with_h0}")
    Hd = G.affine_scan(dev(Az), dev(bz), None if h0 is None else dev(h0), chunk_len=chunk, time_invariant=True)
    H = host(Hd)
    ga, gb, gh0 = G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), None if h0 is None else dev(h0), chunk_len=chunk, time_invariant=True)
    ga, gb = host(ga).astype(np.float64), host(gb).astype(np.float64)
    assert ga.shape == (batch, d, d)
    rep = lambda a_: np.ascontiguousarray(np.broadcast_to(a_[:, None], (batch, T, d, d)))
    per_step, wb, wh0, _ = oracle.affine_scan_backward(rep(Az), bz, Gh, h0=h0, h=H)
    wa = per_step.sum(axis=1)
    mass = np.abs(per_step).sum(axis=1)  # the magnitudes of the T terms of every entry
    want_ti, _, _ = oracle.affine_scan_backward_time_invariant(Az, bz, Gh, h0=h0, h=H)
    assert np.all(np.abs(wa - want_ti) <= 1e-12 * mass + 1e-300)  # (the two orders of summation, against the terms' magnitudes)
    # conditioning, decided by the oracle alone (as for the time-varying pass): probes of half a unit in the last place
    rng = np.random.default_rng(7)
    eta = 2.0 ** -24 if comp == np.float32 else 2.0 ** -53
    rel = 1e-3 if comp == np.float32 else 1e-9
    tiny = 2 * float(np.finfo(comp).tiny)
    tol_a = rel * mass + tiny  # (a sum of T terms of like sign or not: against the sum of their magnitudes)
    tol_b = rel * np.abs(wb) + 1e-3 * rel * np.abs(wb).max(axis=-1, keepdims=True) + tiny
    sens_a, sens_b = np.zeros_like(wa), np.zeros_like(wb)
    pert = lambda z: None if z is None else (z.astype(np.complex128) + eta * rng.standard_normal(z.shape) * np.where(np.isfinite(z.real), 1.0, 0.0))
    for _ in range(2):
        pa, pb, _, _ = oracle.affine_scan_backward(rep(pert(Az)), pert(bz), Gh, h0=pert(h0), h=pert(H))
        sens_a, sens_b = np.maximum(sens_a, np.abs(pa.sum(axis=1) - wa)), np.maximum(sens_b, np.abs(pb - wb))
    well_a, well_b = sens_a <= tol_a / 16, sens_b <= tol_b / 16
    ra = (np.abs(ga - wa) / tol_a)[well_a].max() if well_a.any() else 0.0
    rb = (np.abs(gb - wb) / tol_b)[well_b].max()
    say(f"  worst error / tolerance: grad A {ra:.3g}, grad bias {rb:.3g}; left out as ill conditioned {1 - well_a.mean():.2e} / {1 - well_b.mean():.2e}; "
        f"largest |grad A| / mass {np.max(np.abs(wa) / mass):.3g}")
    assert ra <= 1 and rb <= 1 and well_a.mean() > 0.7 and well_b.mean() > 0.7
    if with_h0:
        gh0 = host(gh0).astype(np.float64)
        assert np.all(np.abs(gh0 - wh0) <= 2e-3 * np.abs(wh0) + 1e-4 * np.abs(wh0).max())


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_scaled_exp_backward(G, oracle, ctype):
    # the states' scaled exponentials and their gradient with the log-scaling constant detached (Section 4.3)
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(81)
    n, d = 1000, 32
    z = oracle.to_goom(si.normal_f32(si.BASE_SEED + 121, 3, n * d).reshape(n, d).astype(comp))
    z.real += rng.uniform(-3000, 3000, (n, 1)).astype(comp)
    z[5, :] = -np.inf  # a vector of zeros
    g = si.normal_f32(si.BASE_SEED + 122, 4, n * d).reshape(n, d).astype(comp)
    scaled = G.scaled_exp(dev(z))
    got = host(G.scaled_exp_backward(scaled, dev(g))).astype(np.float64)
    want = oracle.scaled_exp_backward(z, g)
    rel = 4e-6 if comp == np.float32 else 1e-13  # (the forward values carry their own rounding; the product adds half a unit)
    assert np.all(np.abs(got - want) <= rel * np.abs(want) + 1e-30)
    assert np.all(got[5] == 0)
    top = np.argmax(z.real[0])
    assert abs(abs(got[0, top]) - abs(float(g[0, top])) * math.exp(2.0)) <= 1e-5 * abs(float(g[0, top])) * math.exp(2.0)  # the entry that sets c passes its gradient


@pytest.mark.parametrize("ctype,T,d,chunk", [(np.complex128, 64, 16, 8), (np.complex64, 400, 16, 16), (np.complex64, 300, 32, 0), (np.complex64, 50, 24, 0)])
def test_state_space_layer_forward_and_backward(G, oracle, ctype, T, d, chunk):
    """The recurrent core of the paper's layer (Section 4.3) end to end through the library's calls, forward and backward:
    bias_t = B u_t (an LMME), x_t = A x_{t-1} + bias_t with one matrix for all steps, scaled x_t = exp(x'_t - c + 2) with c
    detached; loss = sum w * scaled.  Every stage against the oracle's, fed the device's forward values."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    batch = 2
    A, _ = si.recurrence_inputs(si.BASE_SEED + 131, batch, 1, d, gain=1.03)
    Az = oracle.to_goom(A[:, 0].astype(comp))
    Bz = oracle.to_goom((si.normal_f32(si.BASE_SEED + 132, 5, batch * d * d).reshape(batch, d, d) / math.sqrt(d)).astype(comp))
    Uz = oracle.to_goom(si.normal_f32(si.BASE_SEED + 133, 6, batch * T * d).reshape(batch, T, d).astype(comp))
    x0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 134, 7, batch * d).reshape(batch, d).astype(comp))
    w = si.normal_f32(si.BASE_SEED + 135, 8, batch * T * d).reshape(batch, T, d).astype(comp)
    say(f"state-space layer T={T} d={d} {np.dtype(ctype).name} chunk={chunk}")
    # forward: rows u_t times B^T
    Btz = np.ascontiguousarray(np.swapaxes(Bz, -1, -2))
    bias_d = G.lmme(dev(Uz), dev(Btz))
    x_d = G.affine_scan(dev(Az), bias_d, dev(x0), chunk_len=chunk, time_invariant=True)
    scaled_d = G.scaled_exp(x_d)
    # backward
    gx_d = G.scaled_exp_backward(scaled_d, dev(w))
    gA, gbias_d, gx0 = G.affine_scan_backward(dev(Az), bias_d, x_d, gx_d, dev(x0), chunk_len=chunk, time_invariant=True)
    gU, gBt = G.lmme_backward(dev(Uz), dev(Btz), bias_d, gbias_d)
    # the oracle's stages on the device's forward values
    bias, x, scaled, gx, gbias = host(bias_d), host(x_d), host(scaled_d), host(gx_d).astype(np.float64), host(gbias_d).astype(np.float64)
    rel = 5e-5 if comp == np.float32 else 1e-11
    want_gx = oracle.scaled_exp_backward(x, w)
    assert np.all(np.abs(gx - want_gx) <= 1e-5 * np.abs(want_gx) + 1e-30)
    rep = np.ascontiguousarray(np.broadcast_to(Az[:, None], (batch, T, d, d)))
    per_step, want_gb, want_gx0, _ = oracle.affine_scan_backward(rep, bias, gx, h0=x0, h=x)
    mass = np.abs(per_step).sum(axis=1)
    err_a = np.abs(host(gA).astype(np.float64) - per_step.sum(axis=1)) / (rel * mass + 1e-30)
    err_b = np.abs(gbias - want_gb) / (rel * np.abs(want_gb) + rel * np.abs(want_gb).max(axis=-1, keepdims=True) + 1e-30)
    want_gU, want_gBt = oracle.lmme_backward(Uz, Btz, gbias, c=bias)
    mU, mBt = oracle.lmme_backward(Uz.real + 0j, Btz.real + 0j, np.abs(gbias), c=bias.real + 0j)
    lrel = 1e-5 if comp == np.float32 else 1e-11
    err_u = np.abs(host(gU).astype(np.float64) - want_gU) / (lrel * mU + 1e-30)
    err_bt = np.abs(host(gBt).astype(np.float64) - want_gBt) / (lrel * mBt + 1e-30)
    say(f"  worst error / tolerance: grad A {err_a.max():.3g}, grad bias {np.median(err_b):.3g} (median) {err_b.max():.3g} (max), "
        f"grad u {err_u.max():.3g}, grad B {err_bt.max():.3g}")
    assert err_a.max() <= 1 and err_u.max() <= 1 and err_bt.max() <= 1
    assert err_b.max() <= 1  # (a contracting or mildly expanding matrix: the adjoints' sums do not cancel; the recurrence's own test covers those that do)
    assert np.all(np.abs(host(gx0).astype(np.float64) - want_gx0) <= 5 * rel * np.abs(want_gx0) + 1e-2 * rel * np.abs(want_gx0).max())
    assert host(gBt).shape == (batch, d, d) and host(gA).shape == (batch, d, d)


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_signed_log_add(G, oracle, ctype):
    comp = np.float32 if ctype == np.complex64 else np.float64
    rng = np.random.default_rng(78)
    n = (1 << 18) + 5
    def gooms(scale):
        z = (rng.normal(0.0, scale, n) + 1j * np.pi * rng.integers(0, 2, n)).astype(ctype)
        z.imag[...] = np.where(z.imag != 0, comp(np.pi), comp(0))
        return z
    x, y = gooms(300.0), gooms(300.0)
    y[:1000] = x[:1000]                      # equal magnitudes: doubling or exact cancellation
    y[1000:2000].real = x[1000:2000].real + comp(1e-3) * rng.standard_normal(1000).astype(comp)  # near cancellation
    x[2000:2010].real = -np.inf              # zero operands
    y[2005:2015].real = -np.inf
    re, sg = oracle.log_add_exp(x, y)
    got = host(G.log_add_exp(dev(x), dev(y)))
    assert np.array_equal(got.imag != 0, sg.astype(bool))
    assert np.all((got.imag == 0) | (got.imag == comp(np.pi)))
    want = re.astype(comp)
    fin = np.isfinite(want)
    assert np.array_equal(np.isneginf(got.real), np.isneginf(want))
    ulp = np.abs(got.real[fin].astype(np.float64) - want[fin].astype(np.float64)) / np.spacing(np.abs(want[fin])).astype(np.float64)
    say(f"log-add {np.dtype(ctype).name}: {np.sum(got.real[fin] != want[fin])} of {fin.sum()} results differ from the rounded oracle, max {ulp.max():.1f} ulp")
    assert ulp.max() <= (1.0 if comp == np.float32 else 4.0)


# (cap: bound on the share of entries the oracle's probes call ill conditioned, about twice what the logs print.  A
# slightly expansive constant matrix makes late states sensitive to the matrix itself: a perturbation of its
# dominant eigenvalue by delta moves a state at step t by t * delta, the same way for every term of the sum.)
@pytest.mark.parametrize("T,d,batch,chunk,ctype,gain,cap", [
    (3000, 32, 3, 0, np.complex64, 1.02, 0.3), (2000, 32, 2, 0, np.complex64, 0.9, 0.05), (500, 16, 2, 7, np.complex64, 1.02, 0.07),
    (100, 8, 2, 9, np.complex64, 1.02, 0.02), (400, 32, 1, 50, np.complex128, 1.02, 0.002), (64, 32, 2, 0, np.complex64, 1.02, 0.02),
    (4100, 32, 1, 1024, np.complex64, 0.9, 0.05), (700, 16, 2, 64, np.complex64, 0.9, 0.05),  # (chunk powers A^L of long and short chunks)
    (600, 64, 2, 0, np.complex64, 1.02, 0.1), (130, 64, 1, 16, np.complex64, 0.9, 0.05)])  # (d = 64: the matrix in registers)
def test_affine_scan_time_invariant(G, oracle, T, d, batch, chunk, ctype, gain, cap):
    # one matrix per sequence, applied at every step (the paper's state-space layer): against the oracle
    # fed the matrix repeated T times
    comp = np.float32 if ctype == np.complex64 else np.float64
    A, b = si.recurrence_inputs(si.BASE_SEED + 57, batch, 1, d, gain=gain)
    A = A[:, 0].astype(comp)  # [batch, d, d]
    _, b = si.recurrence_inputs(si.BASE_SEED + 58, batch, T, d)
    Az, bz = oracle.to_goom(A), oracle.to_goom(b.astype(comp))
    Arep = np.ascontiguousarray(np.broadcast_to(Az[:, None], (batch, T, d, d)))
    say(f"time-invariant recurrence T={T} d={d} batch={batch} chunk={chunk} {np.dtype(ctype).name}")
    # (the conditioning probe perturbs the one matrix that is the input, not T independent copies of it)
    fn = lambda a_, b_, h_: oracle.affine_scan(np.ascontiguousarray(np.broadcast_to(a_[:, None], (batch, T, d, d))), b_, h0=h_, return_kappa=True)
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 59, 9, batch * d).reshape(batch, d).astype(comp))
    for start in (None, h0):
        re, sg, kap, well = with_sensitivity(fn, [Az, bz, start], comp)
        got = host(G.affine_scan(dev(Az), dev(bz), None if start is None else dev(start), chunk_len=chunk, time_invariant=True))
        compare(got, re, sg, kap, name=f"time-invariant T{T}d{d}", max_ill_fraction=cap, well=well)
        # and it is the general entry point's result on the repeated matrix, to rounding
        ref = host(G.affine_scan(dev(Arep), dev(bz), None if start is None else dev(start), chunk_len=chunk))
        same = (ref.imag == got.imag) & (np.abs(ref.real - got.real) <= tolerance(ref.real.astype(np.float64), comp))
        assert same.mean() > 0.98


# ------------------------------------------- shapes beyond the register-resident kernels (up to 1024)

@pytest.mark.parametrize("shape", [(2, 256, 256, 256), (1, 300, 200, 150), (3, 129, 64, 64), (1, 40, 500, 33), (1, 512, 512, 512),
                                   (1, 1024, 1024, 1024), (2, 1000, 130, 1024)])
def test_lmme_large_shapes_complex128(G, oracle, shape):
    """The same passes with double components on the double-precision matrix instruction."""
    from paper_2510_03426_amd import LMME_EXACT
    b, n, d, m = shape
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 64, 5, b * n * d).reshape(b, n, d).astype(np.float64))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 65, 6, b * d * m).reshape(b, d, m).astype(np.float64))
    assert A.dtype == np.complex128
    say(f"large lmme complex128 {shape}")
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B)))
    compare(got, re, sg, kap, name=f"large lmme c128 {shape}", max_ill_fraction=0.002)
    if n * d * m <= 256 ** 3:
        # log-magnitudes N(0, 200^2): the scaled product with its repair pass
        A2, B2 = si.wide_range_goom_pairs(si.BASE_SEED + 66, b, n, d, m, sigma=200.0, dtype=np.complex128)
        re, sg, kap = oracle.lmme(A2, B2, return_kappa=True)
        got = host(G.lmme(dev(A2), dev(B2), flags=LMME_EXACT))
        compare(got, re, sg, kap, name=f"large lmme c128 wide, repaired {shape}", max_ill_fraction=0.002)


@pytest.mark.parametrize("shape", [(2, 256, 256, 256), (1, 300, 200, 150), (3, 129, 64, 64), (1, 40, 500, 33), (1, 512, 512, 512),
                                   (1, 1024, 1024, 1024)])
def test_lmme_large_shapes(G, oracle, shape):
    b, n, d, m = shape
    A = oracle.to_goom(si.normal_f32(si.BASE_SEED + 61, 5, b * n * d).reshape(b, n, d))
    B = oracle.to_goom(si.normal_f32(si.BASE_SEED + 62, 6, b * d * m).reshape(b, d, m))
    say(f"large lmme {shape}")
    re, sg, kap = oracle.lmme(A, B, return_kappa=True)
    got = host(G.lmme(dev(A), dev(B)))
    # (a sum of d Gaussian products falls below 1 / 512 of its mass with probability about 0.05 sqrt(d / 1024))
    compare(got, re, sg, kap, name=f"large lmme {shape}", max_ill_fraction=0.05)
    if n * d * m <= 256 ** 3:
        # log-magnitudes spread over +-60: different rows and columns need very different shifts
        A2, B2 = si.wide_range_goom_pairs(si.BASE_SEED + 63, b, n, d, m, sigma=20.0, dtype=np.complex64)
        re, sg, kap = oracle.lmme(A2, B2, return_kappa=True)
        got = host(G.lmme(dev(A2), dev(B2)))
        # the scaled product is only claimed where its certificate holds: the output's magnitude after the
        # row and column shifts stays 20 + log2(d) bits above the smallest normal float (terms dropped
        # below that level cannot matter)
        ni = np.ceil(A2.real.max(axis=2) * math.log2(math.e))[:, :, None]
        ek = np.ceil(B2.real.max(axis=1) * math.log2(math.e))[:, None, :]
        certified = re * math.log2(math.e) - ni - ek >= -126 + 20 + math.log2(d) + 1
        say(f"  sigma 20: certificate holds for {certified.mean():.2%} of the outputs")
        compare(np.where(certified, got, (re + 1j * np.pi * sg).astype(np.complex64)), re, sg, kap, name=f"large lmme wide {shape}",
                max_ill_fraction=0.05)
        assert certified.mean() > 0.9
        # with the repair pass every output is claimed, also at a spread that leaves nothing certified
        from paper_2510_03426_amd import LMME_EXACT
        got = host(G.lmme(dev(A2), dev(B2), flags=LMME_EXACT))
        compare(got, re, sg, kap, name=f"large lmme wide, repaired {shape}", max_ill_fraction=0.002)
        A3, B3 = si.wide_range_goom_pairs(si.BASE_SEED + 69, b, n, d, m, sigma=200.0, dtype=np.complex64)
        re3, sg3, kap3 = oracle.lmme(A3, B3, return_kappa=True)
        got3 = host(G.lmme(dev(A3), dev(B3), flags=LMME_EXACT))
        compare(got3, re3, sg3, kap3, name=f"large lmme sigma 200, repaired {shape}", max_ill_fraction=0.002)


@pytest.mark.parametrize("T,d,chunk,m,batch", [(24, 256, 0, None, 1), (10, 200, 3, None, 2), (9, 160, 4, 70, 1), (6, 512, 2, None, 1),
                                               (5, 300, 5, 300, 1), (3, 1024, 0, None, 1), (7, 131, 3, 5, 1), (5, 255, 2, 129, 1)])
@pytest.mark.parametrize("comp", [np.float32, np.float64])
def test_scan_large_matrices(G, oracle, T, d, chunk, m, batch, comp):
    say(f"large scan T={T} d={d} chunk={chunk} m={m} batch={batch} {np.dtype(comp).name}")
    Z = oracle.to_goom(si.normal_f32(si.BASE_SEED + 64, 12, batch * T * d * d).reshape(batch, T, d, d).astype(comp))
    init = None
    if m is not None:
        init = oracle.to_goom(si.normal_f32(si.BASE_SEED + 65, 13, batch * d * m).reshape(batch, d, m).astype(comp))
    out = host(G.scan(dev(Z), None if init is None else dev(init), chunk_len=chunk))
    fin = host(G.reduce(dev(Z), None if init is None else dev(init), chunk_len=chunk))
    mm = d if m is None else m
    sample = sorted({0, 1, T // 2, T - 1})
    for b in range(batch):
        st = oracle.ScanStream(d, m=mm, init=None if init is None else init[b], scaled=True)
        re, sg, kap = st.advance(Z[b], sample_t=sample, return_kappa=True)
        # double components: the reference here is itself a double-precision product, good to about
        # kappa sqrt(d) 2^-53; entries are compared up to the kappa that keeps that well inside 1e-10
        klim = None if comp == np.float32 else 2.0 ** 12
        compare(out[b][sample], re, sg, kap, name=f"large scan T{T}d{d} item {b}", max_ill_fraction=0.06, kappa_limit=klim)
        compare(fin[b], re[-1], sg[-1], kap[-1], name=f"large reduce T{T}d{d} item {b}", max_ill_fraction=0.06, kappa_limit=klim)


def test_scan_large_matrices_beyond_double_range(G, oracle):
    # 300 factors of 256 x 256: log-magnitudes pass 830, beyond float and double range
    T, d = 300, 256
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 66, T, d))
    out = G.scan(dev(Z))
    sample = [0, 50, 149, 150, 151, 299]
    re, sg, kap = oracle.ScanStream(d, scaled=True).advance(Z, sample_t=sample, return_kappa=True)
    compare(host(out[sample]), re, sg, kap, name="large scan T300 d256", max_ill_fraction=0.06)
    from scipy.special import digamma
    lam = 0.5 * (math.log(2.0) + digamma(d / 2))
    top = float(host(out[T - 1]).real.max())
    say(f"  log-magnitude of the last prefix {top:.1f}; growth per step {top / T:.4f} (closed form {lam:.4f})")
    assert top > 800 and abs(top / T - lam) < 0.03


def test_caller_stream_and_profile_records(G, oracle):
    # the library enqueues on the caller's stream and never synchronises; per-kernel timings come back by label
    import torch
    from paper_2510_03426_amd import Goom
    T, d = 600, 32
    Z = dev(oracle.to_goom(si.normal_chain(si.BASE_SEED + 67, T, d)))
    want = host(G.scan(Z, chunk_len=50))
    side = torch.cuda.Stream()
    g2 = Goom(0, stream=side)
    with torch.cuda.stream(side):
        out = g2.scan(Z, chunk_len=50)
    side.synchronize()
    assert np.array_equal(host(out).view(np.uint32), want.view(np.uint32))
    g2.set_stream(torch.cuda.default_stream())
    out2 = g2.scan(Z, chunk_len=50)
    assert np.array_equal(host(out2).view(np.uint32), want.view(np.uint32))
    g2.profile_enable(True)
    g2.scan(Z, chunk_len=50)
    recs = g2.profile_records()
    g2.profile_enable(False)
    labels = [l for l, _ in recs]
    assert any("phase1" in l for l in labels) and any("phase3" in l for l in labels) and all(ms >= 0 for _, ms in recs)


def test_scan_replays_from_a_captured_graph(G, oracle):
    # the library allocates nothing, never synchronises and clears nothing with memsets, so a call can be recorded
    # into a HIP graph: three replays on fresh inputs, eager work and synchronisations in between, each against
    # the eager result on the same input
    import torch
    from paper_2510_03426_amd import Goom
    T, d = 700, 64
    zs = [dev(oracle.to_goom(si.normal_chain(si.BASE_SEED + 120 + i, T, d))) for i in range(3)]
    z = torch.empty_like(zs[0])
    out = torch.empty_like(z)
    g2 = Goom(0)
    z.copy_(zs[0])
    g2.scan(z, chunk_len=50, out=out)  # sizes the cached workspace before anything is captured
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g2.set_stream(torch.cuda.current_stream())
        g2.scan(z, chunk_len=50, out=out)
    g2.set_stream(torch.cuda.default_stream())
    for i in (1, 2, 0):
        want = host(G.scan(zs[i], chunk_len=50))
        z.copy_(zs[i])
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        assert np.array_equal(host(out).view(np.uint32), want.view(np.uint32)), f"replay on input {i} differs from the eager scan"


def test_streaming_probes(G, oracle):
    # the measurement aid: copy copies, fill fills, read leaves the data alone (ragged size, not a multiple of the grid)
    import torch
    n = (1 << 20) + 4 * 37
    a = torch.arange(n, dtype=torch.float32, device="cuda")
    b = torch.zeros_like(a)
    G.probe_bandwidth(a, b, 2)
    assert torch.equal(a, b)
    G.probe_bandwidth(a, b, 1)
    assert torch.equal(b.view(-1, 4), torch.tensor([1.0, 2.0, 3.0, 4.0], device="cuda").expand(n // 4, 4))
    keep = b.clone()
    G.probe_bandwidth(a, b, 0)
    assert torch.equal(b, keep) and torch.equal(a, torch.arange(n, dtype=torch.float32, device="cuda"))
    # the matrix-unit probe runs and leaves its sink alone
    sink = torch.zeros(4, device="cuda")
    G.probe_matrix_unit(sink, 8)
    G.probe_matrix_unit(sink, 8, double=True)
    torch.cuda.synchronize()
    assert torch.count_nonzero(sink).item() == 0


# ------------------------------------------------------------------ degenerate cases of the method

@pytest.mark.parametrize("d", [1, 3, 16, 64, 200])
def test_degenerate_chains(G, oracle, d):
    """Zero factors, zero rows and columns, identities, permutations, scalars, single steps: results are
    exact here (no rounding is involved, or the oracle decides), so they are compared exactly or to the
    tolerance, and a zero must come out as (-inf, 0)."""
    rng = np.random.default_rng(90 + d)
    T = 12
    x = si.normal_f32(si.BASE_SEED + 68, 14, T * d * d).reshape(T, d, d).copy()
    # a) identities and permutations only: every prefix is a permutation matrix, exactly
    perm = np.stack([np.eye(d, dtype=np.float32)[rng.permutation(d)] for _ in range(T)])
    out = host(G.scan(dev(oracle.to_goom(perm)), chunk_len=5))
    want = np.eye(d)
    for t in range(T):
        want = perm[t].astype(np.float64) @ want
        assert np.array_equal(np.isneginf(out[t].real), want == 0), (d, t)
        assert np.all(out[t].real[want != 0] == 0.0) and np.all(out[t].imag == 0.0)
    # b) a zero factor in the middle: every later prefix is zero; before it, the oracle's values
    xz = x.copy()
    xz[7] = 0.0
    Z = oracle.to_goom(xz)
    out = host(G.scan(dev(Z), chunk_len=4))
    assert np.all(np.isneginf(out[7:].real)) and np.all(out[7:].imag == 0)
    re, sg, kap = oracle.scan(Z[:7], return_kappa=True)
    compare(out[:7], re, sg, kap, name=f"before the zero factor d{d}", max_ill_fraction=0.05 if d < 4 else 0.06)
    assert np.all(np.isneginf(host(G.reduce(dev(Z), chunk_len=4)).real))
    # c) zero rows and zero columns inside factors (all-zero rows of a tile must not produce NaN)
    xr = x.copy()
    xr[2, d // 2, :] = 0.0
    xr[5, :, 0] = 0.0
    xr[9, d - 1, :] = 0.0
    Z = oracle.to_goom(xr)
    out = host(G.scan(dev(Z), chunk_len=3))
    re, sg, kap = oracle.scan(Z, return_kappa=True)
    assert not np.any(np.isnan(out.real))
    assert np.array_equal(np.isneginf(out.real), np.isneginf(re))
    compare(out, re, sg, kap, name=f"zero rows and columns d{d}", max_ill_fraction=0.05 if d < 4 else 0.08)
    # d) a single step is the matrix itself, bit for bit where it is finite
    Z1 = oracle.to_goom(x[:1])
    one = host(G.scan(dev(Z1)))
    re, sg, kap = oracle.scan(Z1, return_kappa=True)
    compare(one, re, sg, kap, name=f"single step d{d}", max_ill_fraction=0.0)
    # e) LMME with a zero operand, and with the identity on either side
    A = oracle.to_goom(x[0])
    I = oracle.to_goom(np.eye(d, dtype=np.float32))
    Zero = oracle.to_goom(np.zeros((d, d), dtype=np.float32))
    assert np.all(np.isneginf(host(G.lmme(dev(A), dev(Zero))).real)) and np.all(np.isneginf(host(G.lmme(dev(Zero), dev(A))).real))
    for got in (host(G.lmme(dev(A), dev(I))), host(G.lmme(dev(I), dev(A)))):
        assert np.array_equal(got.imag, A.imag) and np.abs(got.real - A.real).max() <= 1e-5 * max(1.0, np.abs(A.real).max())
