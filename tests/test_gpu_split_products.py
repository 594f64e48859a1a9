"""Float products and scans of large matrices in three bf16 parts: sizes around the tiles of both kernels and the inner step, entries whose lower parts lie far
below a row's largest, chunks of every kind, and the workspace that is too small for it."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, compare, dev, host, run_scan_case, tolerance, with_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


def operands(oracle, shape, seed, spread):
    batch, n, d, m = shape
    out = []
    for k, s in ((1, (batch, n, d)), (2, (batch, d, m))):
        z = oracle.to_goom(si.normal_f32(si.BASE_SEED + seed, k, int(np.prod(s))).reshape(s))
        z.real += (np.random.default_rng(seed + k).standard_normal(s) * spread).astype(np.float32)
        out.append(z)
    return out


# inner sizes of one step, odd numbers of steps, a part of one; rows and columns at the edges of 32 and 128; both kernels (few tiles, many)
@pytest.mark.parametrize("shape,spread", [((1, 129, 7, 3), 0), ((2, 1, 300, 1), 0), ((1, 130, 16, 129), 0), ((1, 31, 129, 33), 0), ((1, 257, 145, 65), 0),
                                          ((64, 129, 47, 20), 0), ((40, 150, 33, 131), 0), ((1, 1024, 80, 1024), 0), ((1, 256, 1024, 40), 0),
                                          ((3, 140, 150, 60), 15), ((70, 132, 80, 17), 15), ((1, 129, 200, 33), 20)])
def test_products(G, oracle, shape, spread):  # noqa: F811
    A, B = operands(oracle, shape, 1200 + shape[1] + shape[2], spread)
    if spread:
        A[:, 3] = -np.inf
        B[:, :, 1] = -np.inf
        A[:, 5, 1:] = -np.inf  # a row with one entry
    got = host(G.lmme(dev(A), dev(B)))
    for i in range(min(shape[0], 3)):
        re, sg, kap, well = with_sensitivity(lambda a, b: oracle.lmme(a, b, return_kappa=True), [A[i], B[i]], np.float32, nprobe=1)
        compare(got[i], re, sg, kap, name=f"product {shape}", max_ill_fraction=0.5 if spread else 0.05, well=well)
        # these outputs are one float sum and one logarithm away from exact: sqrt(d) / 2 units of 2^-24 of a sum kappa times its result, the
        # exponentials' (2^-22) and the logarithm's last place
        plain = (kap < 16) & np.isfinite(re) & np.isfinite(got[i].real) & (spread == 0)
        bound = kap * (np.sqrt(shape[2]) * 2.0 ** -24 + 2.0 ** -22) + np.abs(re) * 2.0 ** -22 + 2.0 ** -22
        err = np.abs(got[i].real - re)
        assert np.all(err[plain] <= bound[plain])


# gap: how many powers of two below its row's (A) or column's (B) largest entry, which meets a zero, lies all that counts.  Both kernels (few tiles, many)
@pytest.mark.parametrize("gap_a,gap_b", [(0, 0), (100, 0), (0, 125), (125, 0), (140, 0), (0, 140), (70, 50)])
@pytest.mark.parametrize("batch,n,m", [(1, 129, 40), (40, 140, 131)])
def test_all_bits_of_small_entries(G, oracle, batch, n, m, gap_a, gap_b):  # noqa: F811
    """Three terms a sum: without its operands' third parts (2^-17 of them) it would miss the bound, and without the lift these are lost at gaps above 110."""
    A, B = operands(oracle, (batch, n, 5, m), 1250 + n, 0)
    # (What counts comes out near 1, where the result's last place is 2^-23 or below.  It is a difference of logarithms from its row's largest that is rounded to
    # floats when an operand is converted; one operand's entries lie near 2^-gap for that, the other's as far above 1, and the differences are floats.)
    up = max(gap_a, gap_b)
    level_a, level_b = (-up, up) if gap_a >= gap_b else (up, -up)
    A.real += np.float32(level_a * np.log(2.0))
    B.real += np.float32(level_b * np.log(2.0))
    A[:, :, 0] = np.float32((level_a + gap_a) * np.log(2.0))
    B[:, 0] = -np.inf
    A[:, :, 1] = -np.inf
    B[:, 1] = np.float32((level_b + gap_b) * np.log(2.0))
    got = host(G.lmme(dev(A), dev(B)))
    for i in range(min(batch, 3)):
        re, sg, kap = oracle.lmme(A[i], B[i], return_kappa=True)
        # two exponentials and their corrections (2^-22), the products left out (2^-24), three sums (2^-24 each); the logarithm's last places
        bound = kap * 2.0 ** -21 + (1.0 + np.abs(re)) * 2.0 ** -22
        assert np.all(np.abs(got[i].real - re) <= bound), float((np.abs(got[i].real - re) / bound).max())
        assert np.array_equal(got[i].imag > 1, sg == 1)


@pytest.mark.parametrize("chunk", [1, 2, 5])
@pytest.mark.parametrize("d", [140, 260])
def test_all_bits_in_scans(G, oracle, d, chunk):  # noqa: F811
    """Positive matrices of two entries a row: sums of two terms, without cancellation."""
    T = 5
    Z = np.full((T, d, d), -np.inf, dtype=np.complex64)
    x = si.normal_f32(si.BASE_SEED + 1460 + d, 1, T * d * 2).reshape(T, d, 2)
    i = np.arange(d)
    Z.real[:, i, i], Z.real[:, i, (i + 1) % d] = x[..., 0], x[..., 1]
    re, sg, kap = oracle.scan(Z, return_kappa=True)
    got = host(G.scan(dev(Z), chunk_len=chunk))
    some = re > -np.inf
    assert np.array_equal(some, got.real > -np.inf) and not got[some].imag.any()
    bound = T * 2.0 ** -21 + (1.0 + np.abs(re[some])) * 2.0 ** -22  # (a product as above each step)
    err = np.abs(got.real[some] - re[some])
    assert np.all(err <= bound), float((err / bound).max())


@pytest.mark.parametrize("batch,n,d,m", [(3, 128, 1024, 128), (1, 130, 700, 20), (2, 7, 513, 100)])
def test_products_in_the_room_of_floats(G, oracle, batch, n, d, m):  # noqa: F811
    """A workspace for operands and product in floats: too small for three parts of the operands where the inner dimension is long."""
    import ctypes as C
    import torch
    A, B = operands(oracle, (batch, n, d, m), 1270 + n, 0)
    pad = lambda v, k: -(-v // k) * k
    up = lambda v: pad(v, 256)
    N, M, K = pad(n, 128), pad(m, 128), pad(d, 16)
    room = up(batch * N * K * 4) + up(batch * N * 4) + up(batch * M * K * 4) + up(batch * M * 4) + up(batch * M * N * 4)
    z, w, out = dev(A), dev(B), dev(np.zeros((batch, n, m), dtype=np.complex64))
    ws = torch.empty(room, dtype=torch.uint8, device="cuda")
    run = lambda size: G.lib.goom_lmme(G._ctx, *(C.c_void_p(t.data_ptr()) for t in (z, w, out)), batch, n, d, m, 0, 0, C.c_void_p(ws.data_ptr()), size)
    assert run(room) == 0
    for i in range(batch):
        re, sg, kap, well = with_sensitivity(lambda a, b: oracle.lmme(a, b, return_kappa=True), [A[i], B[i]], np.float32, nprobe=1)
        compare(host(out)[i], re, sg, kap, name=f"product in floats {n}", max_ill_fraction=0.05, well=well)
    least = min(room, G.lib.goom_lmme_workspace_bytes(batch, n, d, m, 0, 0))
    assert run(least) == 0 and run(least - 256) != 0


# room: what these calls asked for with all products in floats
@pytest.mark.parametrize("batch,n,d,m,room", [(3, 128, 128, 1024, 13593600), (2, 64, 200, 700, 8040448)])
def test_products_backward_in_the_room_of_floats(G, oracle, batch, n, d, m, room):  # noqa: F811
    import ctypes as C
    import torch
    A, B = (dev(v) for v in operands(oracle, (batch, n, d, m), 1275 + n, 0))
    P = G.lmme(A, B)
    Gc = dev(si.normal_f32(si.BASE_SEED + 1276, 3, batch * n * m).reshape(batch, n, m))
    want = G.lmme_backward(A, B, P, Gc)
    assert room < G.lib.goom_lmme_backward_workspace_bytes(batch, n, d, m, 0, 0)
    ws, got = torch.empty(room, dtype=torch.uint8, device="cuda"), [torch.empty_like(v) for v in want]
    run = lambda size: G.lib.goom_lmme_backward(G._ctx, *(C.c_void_p(t.data_ptr()) for t in (A, B, P, Gc, *got)), batch, n, d, m, 0, 0, C.c_void_p(ws.data_ptr()), size)
    assert run(room) == 0
    for g, w in zip(got, want):
        assert np.linalg.norm(host(g) - host(w)) <= 1e-5 * np.linalg.norm(host(w))
    assert run(room // 2) != 0


@pytest.mark.parametrize("T,d,m,batch,room", [(6, 200, 5, 1, 8686080), (12, 130, 130, 1, 30937856)])
def test_scan_backward_in_the_room_of_floats(G, oracle, T, d, m, batch, room):  # noqa: F811
    import ctypes as C
    import torch
    z = dev(np.stack([oracle.to_goom(si.normal_chain(si.BASE_SEED + 1680 + i, T, d)) for i in range(batch)]))
    S0 = dev(oracle.to_goom(si.normal_f32(si.BASE_SEED + 1690, 1, batch * d * m).reshape(batch, d, m)))
    P = G.scan(z, S0)
    Gp = dev(si.normal_f32(si.BASE_SEED + 1691, 1, batch * T * d * m).reshape(batch, T, d, m))
    want = G.scan_backward(z, P, Gp, S0)
    full = G.lib.goom_scan_backward_workspace_bytes(T, d, m, batch, 0, None, 1)
    assert room < full
    ws, got = torch.empty(full, dtype=torch.uint8, device="cuda"), [torch.empty_like(v) for v in want]
    run = lambda size: G.lib.goom_scan_backward(G._ctx, *(C.c_void_p(t.data_ptr()) for t in (z, S0, P, Gp, *got)), T, d, m, batch, 0, None, C.c_void_p(ws.data_ptr()), size)
    assert run(full - 256) == 0  # (two converted matrices a chunk)
    assert all(np.array_equal(host(g), host(w)) for g, w in zip(got, want))
    assert run(room) == 0
    for g, w in zip(got, want):  # (other products, other chunks: sums of d terms that cancel, over T steps)
        assert np.linalg.norm(host(g) - host(w)) <= 1e-3 * np.linalg.norm(host(w))
    assert run(room // 2) != 0


# chunks of one step, of two, uneven ones (the last shorter: identities), a single one; states of their own width; several items
@pytest.mark.parametrize("T,d,chunk,m,batch", [(5, 257, 1, None, 1), (7, 300, 2, None, 2), (8, 260, 3, 20, 1), (6, 130, 6, None, 2), (9, 200, 4, 300, 1), (5, 100, 2, 140, 1),
                                               (11, 140, 0, None, 1), (1, 270, 0, None, 1), (2, 384, 0, 1, 3)])
def test_scans(G, oracle, T, d, chunk, m, batch):  # noqa: F811
    run_scan_case(G, oracle, T, d, chunk, m=m, batch=batch, seed=1300 + d, name=f"in parts d={d} m={m}")


def test_scan_of_rows_far_apart(G, oracle):  # noqa: F811
    T, d = 6, 264
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 1400, T, d))
    Z.real += (np.linspace(-40, 40, d)[:, None] - np.linspace(-40, 40, d)[None, :]).astype(np.float32)  # units of their own: D A D^-1
    Z[2] += np.float32(2000.0)
    Z[3, 7] = -np.inf
    re, sg, kap, well = with_sensitivity(lambda z: oracle.scan(z, return_kappa=True), [Z], np.float32, nprobe=2)
    for chunk in (2, 6):
        compare(host(G.scan(dev(Z), chunk_len=chunk)), re, sg, kap, name=f"far apart chunk={chunk}", max_ill_fraction=0.05, well=well)


def whole_power(x):
    """The first float from x on that is a float's power of two to a quarter (the conversion corrects the product with log2(e) by no more than a few units)."""
    x = np.float32(x)
    while abs(float(x) * np.log2(np.e) - float(np.float32(float(x) * np.log2(np.e)))) > 0.25:
        x = np.nextafter(x, np.float32(np.inf))
    return float(x)


# (log-magnitudes whose last place is 128 and more: the factors' entries are all alike, and so are the states', whose sums are of one sign)
@pytest.mark.parametrize("reduce", [False, True])
@pytest.mark.parametrize("T,d,m,chunk", [(6, 140, None, 2), (5, 300, 3, 1), (7, 270, None, 7), (9, 260, None, 0)])
@pytest.mark.parametrize("magnitude", [2.0e9, -2.0e9, 3.0e12])
def test_magnitudes_of_any_size(G, T, d, m, chunk, magnitude, reduce):  # noqa: F811
    step = whole_power(magnitude)
    Z = np.full((1, T, d, d), step, dtype=np.complex64)
    Z[0, 1, 5] = -np.inf
    init = None if m is None else dev(np.full((1, d, m), -step, dtype=np.complex64))
    if reduce:
        got = host(G.reduce(dev(Z), init, chunk_len=chunk))[:, None]
    else:
        got = host(G.scan(dev(Z), init, chunk_len=chunk))
    first = T if reduce else 1
    want = np.arange(first, T + 1) * step - (0.0 if m is None else step)
    assert not got[got.real > -np.inf].imag.any()
    for i, w in enumerate(want):
        z = got[0, i].real
        if first + i == 2:  # the empty row's own step
            assert np.all(z[5] == -np.inf)
            z = np.delete(z, 5, axis=0)
        # a rounding of each factor's shift and of the state's logarithm
        assert np.abs(z - w).max() <= 2.0 ** -22 * T * abs(step), (first + i, z.min(), z.max(), w)


@pytest.mark.parametrize("chunk", [2, 6, 1])
@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("d", [200, 300])
def test_entries_that_are_not_finite_show(G, oracle, d, value, chunk):  # noqa: F811
    """In the row that they lie in, and in every state from the next step on; but a NaN above 256 counts as zero, as in all large products."""
    T = 6
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 1450, T, d))
    Z.real[2, 3, 4] = value
    if d > 256 and value != value:
        got = host(G.scan(dev(Z[None]), chunk_len=chunk))
        Z.real[2, 3, 4] = -np.inf
        assert np.array_equal(got, host(G.scan(dev(Z[None]), chunk_len=chunk)))
        return
    failed = [(z != z) | (z == np.inf) for z in host(G.scan(dev(Z[None]), chunk_len=chunk))[0].real]
    assert not np.any(failed[:2]) and np.all(failed[2][3]) and not np.any(np.delete(failed[2], 3, axis=0)) and np.all(failed[3:])


def test_more_matrices_than_a_grid_is_high(G, oracle):  # noqa: F811
    """Chunks of two steps whose matrices are all converted ahead: up to twice as many as the chains, which are at most 65535."""
    batch, T, d, m = 33000, 2, 2, 260
    z = dev(oracle.to_goom(si.normal_chain(si.BASE_SEED + 1470, batch * T, d)).reshape(batch, T, d, d))
    init = dev(oracle.to_goom(si.normal_f32(si.BASE_SEED + 1471, 1, batch * d * m).reshape(batch, d, m)))
    got = host(G.scan(z, init, chunk_len=T))
    half = batch // 2  # (as many 128 x 128 tiles as fill the chip by far: the same kernels)
    for part in (slice(0, half), slice(half, batch)):
        assert np.array_equal(got[part].view(np.uint32), host(G.scan(z[part], init[part], chunk_len=T)).view(np.uint32))
    for i in (0, batch - 1):
        re, sg, kap, well = with_sensitivity(lambda a, b: oracle.scan(a, init=b, return_kappa=True), [host(z[i]), host(init[i])], np.float32, nprobe=1)
        compare(got[i], re, sg, kap, name=f"item {i}", max_ill_fraction=0.05, well=well)


def launches_of(G, run):  # noqa: F811
    """How much a call enqueues: the nodes of the graph that it is captured into."""
    import ctypes as C
    import torch
    run()  # (sizes the workspace)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        G.set_stream(torch.cuda.current_stream())
        run()
    G.set_stream(torch.cuda.default_stream())
    n = C.c_size_t()
    assert G.lib.hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(n)) == 0
    return n.value


def test_items_share_launches(G, oracle):  # noqa: F811
    T, d, m = 3, 130, 4
    count = []
    for batch in (2, 20):
        z = dev(np.stack([oracle.to_goom(si.normal_chain(si.BASE_SEED + 1480 + i, T, d)) for i in range(batch)]))
        init = dev(oracle.to_goom(si.normal_f32(si.BASE_SEED + 1490, 1, batch * d * m).reshape(batch, d, m)))
        out = dev(np.zeros((batch, T, d, m), dtype=np.complex64))
        count.append(launches_of(G, lambda: G.scan(z, init, chunk_len=T, out=out)))
    assert count[0] == count[1] > 0


def test_static_scratch(G, oracle):  # noqa: F811
    import torch
    for T, d in ((4, 300), (24, 300), (12, 520)):  # beside the room for it, and too large for that
        z = dev(oracle.to_goom(si.normal_chain(si.BASE_SEED + 1500 + d, T, d)))
        out = torch.empty_like(z)
        G.scan_static(z, out)
        ref = G.scan(z)
        torch.cuda.synchronize()
        a, b = host(out), host(ref)
        assert np.quantile(np.abs(a.real - b.real), 0.99) < 1e-3


# beside the room for it, too large for that (two converted matrices a chunk, longer chunks, one chunk), and too large for the products in parts
@pytest.mark.parametrize("T,d,batch,chunk", [(4, 300, 1, 0), (24, 300, 1, 0), (12, 520, 1, 0), (60, 300, 1, 0), (6, 520, 1, 3), (3, 520, 4, None)])
def test_static_scratch_bits(G, oracle, T, d, batch, chunk):  # noqa: F811
    import torch
    z = np.stack([oracle.to_goom(si.normal_chain(si.BASE_SEED + 1500 + d + i, T, d)) for i in range(batch)])
    out = torch.empty_like(dev(z))
    G.scan_static(dev(z), out, chunk_len=chunk or 0)
    got = host(out)
    same = lambda L: np.array_equal(got.view(np.uint32), host(G.scan(dev(z), chunk_len=L)).view(np.uint32))
    if chunk is None:  # the float products: as good as the others, not their bits
        assert not any(same(L) for L in (0, 8, 16, 32))
        re, sg, kap, well = with_sensitivity(lambda a: oracle.scan(a, return_kappa=True), [z[-1]], np.float32, nprobe=1)
        compare(got[-1], re, sg, kap, name=f"static scratch {T} x {d}", max_ill_fraction=0.05, well=well)
    else:
        assert same(chunk) or any(same(L) for L in (8, 16, 32, 64))


@pytest.mark.parametrize("T,d,m,chunk", [(7, 300, None, 3), (6, 270, 5, 6), (9, 384, None, 5), (7, 140, 200, 3)])
def test_scans_with_room_for_two_matrices_a_chunk(G, oracle, T, d, m, chunk):  # noqa: F811
    """Matrices converted step by step, in both phases: the same bits."""
    import ctypes as C
    import torch
    from paper_2510_03426_amd.binding import ScanOpts
    batch, opts = 2, ScanOpts(chunk, 0)
    z = dev(np.stack([oracle.to_goom(si.normal_chain(si.BASE_SEED + 1600 + d + i, T, d)) for i in range(batch)]))
    init = None if m is None else dev(oracle.to_goom(si.normal_f32(si.BASE_SEED + 1610, 1, batch * d * m).reshape(batch, d, m)))
    cols = m or d
    for final in (False, True):
        size = G.lib.goom_reduce_workspace_bytes if final else G.lib.goom_scan_workspace_bytes
        call = G.lib.goom_reduce if final else G.lib.goom_scan
        want = host((G.reduce if final else G.scan)(z, init, chunk_len=chunk))
        full = size(T, d, cols, batch, 0, C.byref(opts))
        out = dev(np.zeros(want.shape, dtype=np.complex64))
        ws = torch.full((full,), 255, dtype=torch.uint8, device="cuda")  # (what is not written reads as NaN)
        p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
        assert call(G._ctx, p(z), p(init), p(out), T, d, cols, batch, 0, C.byref(opts), p(ws), full - 256) == 0
        assert np.array_equal(host(out).view(np.uint32), want.view(np.uint32))
