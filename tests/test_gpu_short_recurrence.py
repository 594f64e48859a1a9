"""The recurrence over few tokens, in chunks shorter than a plain scan's: lengths at the rule's edges against the oracle, and a workspace with room for
the longer chunks alone."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2510_03426_amd.binding import ScanOpts
from test_gpu_parity import G, compare, dev, host, say, with_sensitivity  # noqa: F401
from test_gpu_vector_chains import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [5, 16, 32, 64, 65, 128])
def test_short_sequences(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, batch in ((23, 1), (24, 2), (28, 1), (59, 1), (300, 1), (589, 1), (787, 1)):
        if T * d * d > 1300000:
            continue
        Az, bz, h0 = inputs(oracle, 1400 + d, batch, T, d, ctype, False)
        say(f"short recurrence T={T} d={d} batch={batch} {np.dtype(ctype).name}")
        fn = lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True)
        re, sg, kap, well = with_sensitivity(fn, [Az, bz, h0], comp, nprobe=3)
        got = host(G.affine_scan(dev(Az), dev(bz), dev(h0)))
        compare(got, re, sg, kap, name=f"T{T}d{d}", max_ill_fraction=0.25, well=well)


@pytest.mark.parametrize("ctype,T,d,batch", [(np.complex64, 28, 8, 1), (np.complex64, 31, 64, 1), (np.complex64, 24, 100, 1), (np.complex64, 31, 128, 2),
                                             (np.complex128, 24, 8, 1), (np.complex128, 31, 16, 2)])
def test_units_of_their_own(G, oracle, ctype, T, d, batch):  # noqa: F811
    """D A D^-1, D b and D h0, D over e^+-30 (e^+-250), forward and backward: one chunk, without products whose columns would have to share an exponent."""
    comp, span = (np.float32, 30) if ctype == np.complex64 else (np.float64, 250)
    units = np.random.default_rng(d).permutation(np.linspace(-span, span, d)).astype(comp)
    Az, bz, h0 = inputs(oracle, 1470 + d, batch, T, d, ctype, False)
    Az.real += units[:, None] - units[None, :]
    bz.real += units
    h0.real += units
    re, sg, kap, well = with_sensitivity(lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True), [Az, bz, h0], comp, nprobe=2)
    H = host(G.affine_scan(dev(Az), dev(bz), dev(h0)))
    compare(H, re, sg, kap, name=f"units T{T}d{d}", max_ill_fraction=0.25, well=well)
    Gh = np.random.default_rng(T + d).normal(size=H.shape).astype(comp)
    got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), dev(H), dev(Gh), dev(h0))]
    for name, g, w in zip(("A", "bias", "h0"), got, oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)[:3]):
        # (as below)
        assert np.linalg.norm(g - w) <= (1e-3 if comp == np.float32 else 1e-10) * np.linalg.norm(w), (name, np.linalg.norm(g - w) / np.linalg.norm(w))


@pytest.mark.parametrize("ctype,T,d", [(np.complex64, 32, 64), (np.complex64, 47, 100), (np.complex64, 40, 8), (np.complex128, 47, 12)])
def test_two_chunks_in_units_of_their_own(G, oracle, ctype, T, d):  # noqa: F811
    """Between two chunks nothing passes but a vector: from zero the states, and always the adjoints, need no chunk's product."""
    comp, span = (np.float32, 30) if ctype == np.complex64 else (np.float64, 250)
    units = np.random.default_rng(d).permutation(np.linspace(-span, span, d)).astype(comp)
    Az, bz, h0 = inputs(oracle, 1480 + d, 1, T, d, ctype, False)
    Az.real += units[:, None] - units[None, :]
    bz.real += units
    h0.real += units
    re, sg, kap, well = with_sensitivity(lambda a_, b_: oracle.affine_scan(a_, b_, return_kappa=True), [Az, bz], comp, nprobe=2)
    compare(host(G.affine_scan(dev(Az), dev(bz))), re, sg, kap, name=f"units, from zero, T{T}d{d}", max_ill_fraction=0.25, well=well)
    re, sg = oracle.affine_scan(Az, bz, h0=h0)
    H = (re + 1j * np.pi * sg).astype(ctype)
    Gh = np.random.default_rng(T + d).normal(size=H.shape).astype(comp)
    got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), dev(H), dev(Gh), dev(h0))]
    for name, g, w in zip(("A", "bias", "h0"), got, oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)[:3]):
        assert np.linalg.norm(g - w) <= (1e-3 if comp == np.float32 else 1e-10) * np.linalg.norm(w), (name, np.linalg.norm(g - w) / np.linalg.norm(w))


@pytest.mark.parametrize("T", [28, 31])
def test_logarithms_of_16_rows(G, oracle, T):  # noqa: F811
    """One chunk, whose logarithms are taken of mantissas below 1: a last place of 2^-24 there, and one of the result's (the chunks' own walk: 2^-20)."""
    Az, bz, h0 = inputs(oracle, 1460, 8, T, 16, np.complex64, False)
    re = oracle.affine_scan(Az, bz, h0=h0, return_kappa=True)[0]
    got = host(G.affine_scan(dev(Az), dev(bz), dev(h0)))
    assert np.median(np.abs(got.real - re)) <= 2.0 ** -22 * max(1.0, np.median(np.abs(re)))


@pytest.mark.parametrize("d,former", [(64, 20), (24, 9)])
def test_in_the_room_of_longer_chunks(G, oracle, d, former):  # noqa: F811
    T, batch = 60, 3
    Az, bz, h0 = (dev(v) for v in inputs(oracle, 1490, batch, T, d, np.complex64, False))
    size = lambda chunk: G.lib.goom_affine_scan_workspace_bytes(T, d, batch, 0, C.byref(ScanOpts(chunk, 0)))
    small = size(former)
    assert small < size(0)
    ws, out = torch.empty(small, dtype=torch.uint8, device="cuda"), torch.empty_like(bz)
    run = lambda n: G.lib.goom_affine_scan(G._ctx, *(C.c_void_p(t.data_ptr()) for t in (Az, bz, h0, out)), T, d, batch, 0, C.byref(ScanOpts(0, 0)),
                                           C.c_void_p(ws.data_ptr()), n)
    assert run(small) == 0
    assert np.array_equal(host(out), host(G.affine_scan(Az, bz, h0, chunk_len=former)))
    assert run(small - 256) != 0


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [5, 16, 32, 64, 65, 128])
def test_short_sequences_backward(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, batch in ((23, 1), (24, 2), (59, 1), (300, 1), (517, 1), (589, 1), (787, 1)):
        if T * d * d > 1300000:
            continue
        Az, bz, h0 = inputs(oracle, 1450 + d, batch, T, d, ctype, False)
        H = host(G.affine_scan(dev(Az), dev(bz), dev(h0)))
        want, _ = oracle.scaled_exp(H)
        Gh = (np.random.default_rng(1451 + d + T).normal(size=want.shape) * want).astype(comp)  # as a layer asks for them, from the scaled states
        say(f"short recurrence backward T={T} d={d} batch={batch} {np.dtype(ctype).name}")
        got = [host(v).astype(np.float64) for v in G.affine_scan_backward(dev(Az), dev(bz), dev(H), dev(Gh), dev(h0))]
        for name, g, w in zip(("A", "bias", "h0"), got, oracle.affine_scan_backward(Az, bz, Gh, h0=h0, h=H)[:3]):
            # (as for one matrix: some hundred roundings of a sum's terms, which cancel up to tenfold)
            assert np.linalg.norm(g - w) <= (1e-3 if comp == np.float32 else 1e-10) * np.linalg.norm(w), (name, np.linalg.norm(g - w) / np.linalg.norm(w))


@pytest.mark.parametrize("d,former", [(64, 20), (16, 20)])
def test_backward_in_the_room_of_longer_chunks(G, oracle, d, former):  # noqa: F811
    T, batch = 60, 3
    Az, bz, h0 = (dev(v) for v in inputs(oracle, 1495, batch, T, d, np.complex64, False))
    H = G.affine_scan(Az, bz, h0)
    Gh = G.scaled_exp(H)
    size = lambda chunk: G.lib.goom_affine_scan_backward_workspace_bytes(T, d, batch, 0, C.byref(ScanOpts(chunk, 0)))
    small = size(former)
    assert small < size(0)
    want = G.affine_scan_backward(Az, bz, H, Gh, h0, chunk_len=former)
    ws, out = torch.empty(small, dtype=torch.uint8, device="cuda"), [torch.empty_like(v) for v in want]
    run = lambda n: G.lib.goom_affine_scan_backward(G._ctx, *(C.c_void_p(t.data_ptr()) for t in (Az, bz, h0, H, Gh, *out)), T, d, batch, 0, C.byref(ScanOpts(0, 0)),
                                                    C.c_void_p(ws.data_ptr()), n)
    assert run(small) == 0
    assert all(np.array_equal(host(a), host(b)) for a, b in zip(out, want))
    assert run(small - 256) != 0
