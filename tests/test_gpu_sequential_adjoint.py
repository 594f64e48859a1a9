"""Backward pass of the recurrence over many sequences of d = 32, walked whole: lengths around the rounds in which steps are loaded
(sixteen for the matrices, eight for the chain), zeros among the entries, steps that change every magnitude at once, an initial state or none; against the oracle on
the device's forward states."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, dev, host, say  # noqa: F401
from test_gpu_vector_chains import inputs

pytestmark = pytest.mark.gpu

D, BATCH = 32, 96


@pytest.mark.parametrize("with_h0", [True, False])
@pytest.mark.parametrize("spread", [0.0, 300.0])
@pytest.mark.parametrize("T", [36, 39, 40, 41, 48, 79, 80, 81])
def test_adjoint_walked_whole(G, oracle, T, spread, with_h0):  # noqa: F811
    Az, bz, h0 = inputs(oracle, 500 + T, BATCH, T, D, np.complex64, False)
    # state t in units of e^unit[t]: factors, biases and states far outside float range, gradients not
    unit = np.rint(np.random.default_rng(T).uniform(-spread, spread, (BATCH, T + 1, 1))).astype(np.float32)
    Az.real += (unit[:, 1:] - unit[:, :-1])[..., None]
    bz.real += unit[:, 1:]
    h0.real += unit[:, 0]
    h0 = h0 if with_h0 else None
    put = lambda v: None if v is None else dev(v)
    say(f"adjoint walked whole T={T} spread={spread} h0={with_h0}")
    Hd = G.affine_scan(dev(Az), dev(bz), put(h0))
    H = host(Hd)
    Gh = si.normal_f32(si.BASE_SEED + 501, 10, BATCH * T * D).reshape(BATCH, T, D)
    Gh[:, T // 2] = 0.0
    G.profile_enable(True)
    got = G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), put(h0))
    labels = [k for k, _ in G.profile_records()]
    G.profile_enable(False)
    assert "affine_sequential_adjoint" in labels, labels
    got = [None if v is None else host(v).astype(np.float64) for v in got]
    want = oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)[:3]
    # what half-unit perturbations of the inputs move by more than 1/16 of the tolerance is left out (sums that cancel)
    rng = np.random.default_rng(5)
    pert = lambda z: None if z is None else z.astype(np.complex128) + 2.0 ** -24 * rng.standard_normal(z.shape) * np.isfinite(z.real)
    sens = [None if w is None else np.zeros_like(w) for w in want]
    for _ in range(4):
        probe = oracle.affine_scan_backward(pert(Az), pert(bz), Gh, h0=pert(h0), h=pert(H))[:3]
        sens = [None if w is None else np.maximum(s, np.abs(p - w)) for s, p, w in zip(sens, probe, want)]
    for name, g, w, s in zip(("A", "bias", "h0"), got, want, sens):
        if w is None:
            continue
        assert np.isfinite(g).all(), name
        tol = 1e-3 * np.abs(w) + 1e-6 * np.abs(w).max(axis=tuple(range(1, w.ndim)), keepdims=True) + 2 * float(np.finfo(np.float32).tiny)
        well = s <= tol / 16
        worst = (np.abs(g - w) / tol)[well].max()
        say(f"  {name}: worst error / tolerance {worst:.3g}, left out {1 - well.mean():.2e}")
        assert worst <= 1 and well.mean() > 0.9, (name, worst, well.mean())
    if not with_h0:
        assert np.all(got[0][:, 0] == 0)  # the first matrix multiplies a zero vector


def test_what_is_not_finite_passes_no_gradient(G, oracle):  # noqa: F811
    """A NaN or an infinity in one sequence: its own gradient is zero or infinite, never a NaN, and the other sequences do not see it."""
    T = 40
    Az, bz, h0 = inputs(oracle, 600, BATCH, T, D, np.complex64, False)
    Gh = si.normal_f32(si.BASE_SEED + 601, 10, BATCH * T * D).reshape(BATCH, T, D)
    Hd = G.affine_scan(dev(Az), dev(bz), dev(h0))
    ref = [host(v) for v in G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), dev(h0))]
    H = host(Hd)
    Az[3, 20, 5, 7], bz[4, 11, 2], h0[5, 1] = np.nan, np.nan, np.nan
    Az[6, 20, 5, 7], bz[7, 11, 2], h0[8, 1] = np.inf, np.inf, np.inf
    H[9, 30, 4] = np.nan
    got = [host(v) for v in G.affine_scan_backward(dev(Az), dev(bz), dev(H), dev(Gh), dev(h0))]
    assert not np.isnan(got[0]).any() and not np.isnan(got[1]).any()
    assert got[0][3, 20, 5, 7] == 0 and got[1][4, 11, 2] == 0 and np.all(got[0][5, 0, :, 1] == 0)
    rest = [i for i in range(BATCH) if not 3 <= i <= 9]
    for g, r in zip(got, ref):
        assert np.array_equal(g[rest], r[rest])
