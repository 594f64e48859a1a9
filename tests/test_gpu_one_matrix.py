"""The recurrence with one matrix for all steps, sixteen chunks a workgroup: matrices at and beside the kernel's sizes, a last chunk of one
step and of all, groups of chunks, both directions; the call's sequences at both ends against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import synthetic_inputs as si
from paper_2510_03426_amd.binding import AFFINE_TIME_INVARIANT, ScanOpts
from test_gpu_parity import G, compare, dev, host, say, tolerance, with_sensitivity  # noqa: F401
from test_gpu_vector_chains import inputs

pytestmark = pytest.mark.gpu


# (17, 31, 32: with 32768 steps and more of all sequences; 49 steps: the shortest sequence in chunks; 4099: more chunks than one chain carries)
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d,T,batch", [(17, 241, 136), (31, 512, 65), (32, 1025, 32), (32, 513, 160), (33, 49, 3), (48, 517, 2), (63, 257, 2), (64, 512, 3),
                                       (64, 530, 129), (64, 4099, 1), (65, 50, 2), (100, 128, 2), (127, 513, 1), (128, 63, 2), (128, 528, 1)])
def test_one_matrix_chunks_side_by_side(G, oracle, d, T, batch, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    Az, bz, h0 = inputs(oracle, 900 + d, batch, T, d, ctype, True)
    say(f"one matrix T={T} d={d} batch={batch} {np.dtype(ctype).name}")
    ends = [0, batch - 1] if batch > 1 else [0]
    A2, b2, h2 = (np.ascontiguousarray(v[ends]) for v in (Az, bz, h0))
    rep = lambda a: np.broadcast_to(a[:, None], (len(ends), T, d, d))
    fn = lambda a_, b_, h_: oracle.affine_scan(rep(a_), b_, h0=h_, return_kappa=True)
    re, sg, kap, well = with_sensitivity(fn, [A2, b2, h2], comp, nprobe=3)
    Hd = G.affine_scan(dev(Az), dev(bz), dev(h0), time_invariant=True)
    H = host(Hd)
    compare(H[ends], re, sg, kap, name=f"T{T}d{d}", max_ill_fraction=0.25, well=well, max_out_fraction=1e-4, hard_factor=10.0)
    # the scaled states are those of the states
    sc, c = (host(v).astype(np.float64) for v in G.affine_scan_scaled(dev(Az), dev(bz), dev(h0), time_invariant=True, want_logscale=True))
    want, cw = oracle.scaled_exp(H)
    top = np.abs(want).max(axis=-1, keepdims=True)
    eps = np.finfo(comp).eps
    # (the log's half unit of both sides, on results of at most e^2)
    size = np.maximum(np.abs(np.where(np.isfinite(H.real), H.real, 0)).max(axis=-1, keepdims=True), 16.0)
    assert np.all(np.abs(sc - want) <= 4 * eps * size * top) and np.all(np.abs(c - cw) <= 4 * eps * size[..., 0])
    # gradients as a layer asks for them, from the scaled states
    Gh = (si.normal_f32(si.BASE_SEED + 901, 10, batch * T * d).reshape(batch, T, d) * want).astype(comp)
    got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), Hd, dev(Gh), dev(h0), time_invariant=True)]
    ref = oracle.affine_scan_backward_time_invariant(A2, b2, Gh[ends], h0=h2, h=H[ends])[:3]
    for name, g, w in zip(("A", "bias", "h0"), got, ref):
        assert np.linalg.norm(g[ends] - w) <= (1e-3 if comp == np.float32 else 1e-10) * np.linalg.norm(w), (name, np.linalg.norm(g[ends] - w) / np.linalg.norm(w))


@pytest.mark.parametrize("d", [32, 64, 100])
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_one_matrix_zeros_and_lone_biases(G, d, ctype):  # noqa: F811
    """Zero states, a bias after zeros, terms that cancel and leave a bias below or above their last place, in many chunks."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    T, batch = 600, 64
    none, pi = -np.inf, float(comp(np.pi))
    below, above = (-150.0, -60.0) if comp == np.float32 else (-900.0, -600.0)
    A = np.full((batch, d, d), none, dtype=ctype)
    A[:, 0, 0] = A[:, 1, 1] = 0.0
    A[:, d - 1, 0], A[:, d - 1, 1] = 0.0, 1j * pi  # the last row: h_0 - h_1
    b = np.full((batch, T, d), none, dtype=ctype)
    b[:, 37, 0] = b[:, 37, 1] = 0.0  # (zeros up to there)
    b[:, 50:, d - 1] = below
    b[:, 300:, d - 1] = above
    H = host(G.affine_scan(dev(A), dev(b), time_invariant=True))
    assert np.all(H[:, :37].real == none) and np.all(H[:, 37:, :2] == 0) and np.all(H[:, :, 2:d - 1].real == none)
    assert np.all(H[:, 37:300, d - 1].real == none) and np.abs(H[:, 300:, d - 1].real - above).max() <= 1e-6 * abs(above)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("d", [33, 48, 100])
@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
def test_one_matrix_carries_of_any_exponent(G, d, ctype, sign):  # noqa: F811
    """States that grow (shrink) by e^(3e14) a step, so that the carried vectors' exponents pass 1e15: every chunk starts where the one before ended."""
    comp = np.float32 if ctype == np.complex64 else np.float64
    T, batch, step = 60, 2, float(comp(sign * 3e14))
    A = np.full((batch, d, d), -np.inf, dtype=ctype)
    A[:, range(d), range(d)] = step
    b = np.full((batch, T, d), -np.inf, dtype=ctype)
    h0 = np.zeros((batch, d), dtype=ctype)
    h0[1, ::2] = -np.inf  # (zeros among them stay zeros)
    H = host(G.affine_scan(dev(A), dev(b), dev(h0), time_invariant=True))
    want = np.arange(1, T + 1)[:, None] * step + h0[:, None, :].real
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(H.real), ok) and not H.imag.any()
    # a rounding of the matrix's entry and of the state's logarithm a step
    assert np.abs(H.real[ok] / want[ok] - 1).max() <= 4 * T * np.finfo(comp).eps


# (from zero and of up to 63 steps, or more sequences than fill the chip: one chunk, or two, before the chunks were walked side by side)
@pytest.mark.parametrize("ctype,T,d,batch,from_zero", [(np.complex64, 60, 64, 1, True), (np.complex64, 63, 100, 2, True), (np.complex64, 100, 64, 600, False),
                                                       (np.complex64, 90, 40, 600, False), (np.complex64, 700, 24, 50, False), (np.complex64, 2100, 48, 1, False),
                                                       (np.complex64, 500, 16, 3, False), (np.complex128, 200, 64, 2, False), (np.complex128, 300, 12, 2, False)])
def test_one_matrix_in_units_of_its_own(G, oracle, ctype, T, d, batch, from_zero):  # noqa: F811
    """D A D^-1, D b and D h0, A a rotation and D over e^+-30 (e^+-250), forward and backward: the chunks' product keeps its rows' powers of two."""
    comp, span = (np.float32, 30) if ctype == np.complex64 else (np.float64, 250)
    rng = np.random.default_rng(d + T)
    units = rng.permutation(np.linspace(-span, span, d))
    Q = np.linalg.qr(rng.standard_normal((batch, d, d)))[0]
    Az = (np.log(np.abs(Q)) + units[:, None] - units[None, :] + 1j * np.pi * (Q < 0)).astype(ctype)
    b, h = rng.standard_normal((batch, T, d)), rng.standard_normal((batch, d))
    bz = (np.log(np.abs(b)) + units + 1j * np.pi * (b < 0)).astype(ctype)
    h0 = None if from_zero else (np.log(np.abs(h)) + units + 1j * np.pi * (h < 0)).astype(ctype)
    ends = sorted({0, batch - 1})
    A2, b2, h2 = (None if v is None else np.ascontiguousarray(v[ends]) for v in (Az, bz, h0))
    rep = lambda a: np.broadcast_to(a[:, None], (len(ends), T, d, d))
    re, sg, kap = oracle.affine_scan(rep(A2), b2, h0=h2, return_kappa=True)
    put = lambda v: None if v is None else dev(v)
    got = host(G.affine_scan(dev(Az), dev(bz), put(h0), time_invariant=True))
    # a state in its units: T steps of a rotation, each a rounding of d products of sizes about 1, and of the entries (a float of size 2 span: its last place)
    unit_eps = np.finfo(comp).eps * 2 * span
    g = np.exp(got[ends].real.astype(np.float64) - units) * np.where(got[ends].imag > 1, -1.0, 1.0)
    w = np.exp(re - units) * np.where(sg == 1, -1.0, 1.0)
    assert np.linalg.norm(g - w) <= 4 * T ** 0.5 * unit_eps * np.linalg.norm(w), np.linalg.norm(g - w) / np.linalg.norm(w)
    H = got.copy()
    H[ends] = (re + 1j * np.pi * sg).astype(ctype)
    Gh = (rng.standard_normal(H.shape) * np.exp(H.real - units)).astype(comp)
    got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), dev(H), dev(Gh), put(h0), time_invariant=True)[:2]]
    for name, g, w in zip(("A", "bias"), got, oracle.affine_scan_backward_time_invariant(A2, b2, Gh[ends], h0=h2, h=H[ends])[:2]):
        assert np.linalg.norm(g[ends] - w) <= 4 * T ** 0.5 * unit_eps * np.linalg.norm(w), (name, np.linalg.norm(g[ends] - w) / np.linalg.norm(w))


@pytest.mark.parametrize("d", [48, 64, 100, 128])
def test_one_matrix_rounds_no_more_than_one_chain(G, oracle, d):  # noqa: F811
    """Sixteen chunks as the columns of a product: its sums are of sixteen terms, and these in pairs, as a lane's and sixteen lanes' are in the walk of one chain."""
    T, batch = 192, 4
    rng = np.random.default_rng(d)
    Q = np.linalg.qr(rng.standard_normal((batch, d, d)))[0]
    Az, bz, h0 = (oracle.to_goom(v.astype(np.float32)) for v in (Q, 0.1 * rng.standard_normal((batch, T, d)), rng.standard_normal((batch, d))))
    re, sg = oracle.affine_scan(np.broadcast_to(Az[:, None], (batch, T, d, d)), bz, h0=h0)
    w = np.exp(re) * np.where(sg == 1, -1, 1)
    err = []
    for chunk in (0, T):
        got = host(G.affine_scan(dev(Az), dev(bz), dev(h0), chunk_len=chunk, time_invariant=True))
        err.append(np.linalg.norm(np.exp(got.real.astype(np.float64)) * np.where(got.imag > 1, -1, 1) - w) / np.linalg.norm(w))
    say(f"d={d} in chunks {err[0]:.2e}, one chain {err[1]:.2e}")
    # Roundings of rotations add up as the root of their number: 192 steps on one side, 24 carries and a chunk of eight at most on the other, the last states'
    # ratio 0.41, all states' less.  (Sums of d terms one after the other: 0.46 to 0.66.)
    assert err[0] <= 0.45 * err[1]


def test_one_matrix_in_the_room_of_one_column_walks(G, oracle):  # noqa: F811
    """A workspace too small for the short chunks: longer ones, and the same states and gradients; nothing at all is refused."""
    T, d, batch = 1000, 64, 4
    Az, bz, h0 = (dev(v) for v in inputs(oracle, 990, batch, T, d, np.complex64, True))
    want = G.affine_scan(Az, bz, h0, time_invariant=True)
    size = lambda chunk: G.lib.goom_affine_scan_workspace_bytes(T, d, batch, 0, C.byref(ScanOpts(chunk, AFFINE_TIME_INVARIANT)))
    small = size(32)
    assert small < size(0)
    ws, out = torch.empty(small, dtype=torch.uint8, device="cuda"), torch.empty_like(want)
    run = lambda n: G.lib.goom_affine_scan(G._ctx, *(C.c_void_p(t.data_ptr()) for t in (Az, bz, h0, out)), T, d, batch, 0,
                                           C.byref(ScanOpts(0, AFFINE_TIME_INVARIANT)), C.c_void_p(ws.data_ptr()), n)
    assert run(small) == 0
    torch.cuda.synchronize()
    # (other chunks round differently; 1000 steps of a contraction keep some hundred of a state's roundings)
    assert np.linalg.norm(np.exp(host(out).real) - np.exp(host(want).real)) <= 1e-3 * np.linalg.norm(np.exp(host(want).real))
    assert run(small // 64) != 0
