"""Scans and reductions of few matrices, in chunks shorter than a long chain's: lengths at the rule's edges against the oracle, and a workspace with room
for the longer chunks alone."""
import ctypes as C

import numpy as np
import pytest
import torch

import synthetic_inputs as si
from paper_2510_03426_amd.binding import ScanOpts
from test_gpu_parity import G, compare, dev, host, say, with_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


def chain(oracle, seed, batch, T, d, comp):
    return oracle.to_goom(si.normal_f32(si.BASE_SEED + seed, 3, batch * T * d * d).reshape(batch, T, d, d).astype(comp))


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("d", [5, 16, 31, 64, 65, 128])
def test_short_scans(G, oracle, d, ctype):  # noqa: F811
    comp = np.float32 if ctype == np.complex64 else np.float64
    for T, batch in ((23, 1), (24, 2), (40, 1), (61, 1), (293, 1), (294, 1), (588, 1)):
        if T * d * d > 1300000:
            continue
        z = chain(oracle, 1500 + d + T, batch, T, d, comp)
        say(f"short scan T={T} d={d} batch={batch} {np.dtype(ctype).name}")
        got, last = host(G.scan(dev(z))), host(G.reduce(dev(z)))
        fn = lambda z_: oracle.scan(z_, return_kappa=True)
        for b in range(batch):
            re, sg, kap, well = with_sensitivity(fn, [z[b]], comp, nprobe=3)
            compare(got[b], re, sg, kap, name=f"T{T}d{d}", max_ill_fraction=0.25, well=well)
            compare(last[b], re[-1], sg[-1], kap[-1], name=f"last T{T}d{d}", max_ill_fraction=0.5, well=well[-1])


@pytest.mark.parametrize("comp,T,d,batch", [(np.float32, 24, 40, 1), (np.float32, 31, 64, 1), (np.float32, 24, 100, 1), (np.float32, 31, 128, 2),
                                            (np.float32, 26, 66, 150), (np.float64, 24, 8, 1), (np.float64, 31, 16, 2)])
def test_units_of_their_own(G, oracle, T, d, batch, comp):  # noqa: F811
    """D A D^-1, D over e^+-30 (e^+-250): one chunk, without products whose columns would have to share an exponent."""
    span = 30 if comp == np.float32 else 250
    units = np.random.default_rng(d).permutation(np.linspace(-span, span, d))
    z = chain(oracle, 1585 + d + T, batch, T, d, comp)
    z.real += (units[:, None] - units[None, :]).astype(comp)
    got, last = host(G.scan(dev(z))), host(G.reduce(dev(z)))
    for b in {0, batch - 1}:
        re, sg, kap, well = with_sensitivity(lambda z_: oracle.scan(z_, return_kappa=True), [z[b]], comp, nprobe=2)
        compare(got[b], re, sg, kap, name=f"units T{T}d{d}", max_ill_fraction=0.25, well=well)
        compare(last[b], re[-1], sg[-1], kap[-1], name=f"units, last T{T}d{d}", max_ill_fraction=0.5, well=well[-1])


@pytest.mark.parametrize("d,former", [(64, 20), (100, 20)])
def test_in_the_room_of_longer_chunks(G, oracle, d, former):  # noqa: F811
    T, batch = 60, 3
    z = dev(chain(oracle, 1590, batch, T, d, np.float32))
    size = lambda chunk: G.lib.goom_scan_workspace_bytes(T, d, d, batch, 0, C.byref(ScanOpts(chunk, 0)))
    small = size(former)
    assert small < size(0)
    ws, out = torch.empty(small, dtype=torch.uint8, device="cuda"), torch.empty_like(z)
    run = lambda n: G.lib.goom_scan(G._ctx, C.c_void_p(z.data_ptr()), None, C.c_void_p(out.data_ptr()), T, d, d, batch, 0, C.byref(ScanOpts(0, 0)),
                                    C.c_void_p(ws.data_ptr()), n)
    assert run(small) == 0
    assert np.array_equal(host(out), host(G.scan(z, chunk_len=former)))
    assert run(small - 256) != 0


def test_real_matrices_in_the_room_of_longer_chunks(G):  # noqa: F811
    T, d, former = 60, 100, 20
    x = dev(si.normal_f32(si.BASE_SEED + 1591, 3, T * d * d).reshape(1, T, d, d))
    size = lambda chunk: G.lib.goom_scan_real_workspace_bytes(T, d, d, 1, 0, C.byref(ScanOpts(chunk, 0)))
    small = size(former)
    assert small < size(0)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    out = [torch.empty((1, T, d, d), dtype=torch.complex64, device="cuda") for _ in range(2)]
    run = lambda o, chunk, n: G.lib.goom_scan_real(G._ctx, C.c_void_p(x.data_ptr()), None, C.c_void_p(o.data_ptr()), T, d, d, 1, 0, C.byref(ScanOpts(chunk, 0)),
                                                   C.c_void_p(ws.data_ptr()), n)
    assert run(out[0], 0, small) == 0 and run(out[1], former, small) == 0
    assert np.array_equal(host(out[0]), host(out[1]))
    assert run(out[0], 0, small - 256) != 0
