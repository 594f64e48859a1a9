"""Scans of float chains of every size up to 128, with states of their own width: around the tiles, at the edges of the lanes' groups of four
entries, pairs of small chains of unequal length, zero rows, and matrices that end where their allocation ends."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, compare, dev, host, run_scan_case, say, with_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 17, 18, 19, 21, 30, 31, 33, 34, 47, 49, 50, 62, 63, 65, 66, 79, 81, 97, 113, 126, 127])
def test_square(G, oracle, d):  # noqa: F811
    # several chunks, the last one shorter; two items; grouped carries where that is quick
    run_scan_case(G, oracle, 61, d, 8, batch=2, seed=400 + d, name=f"other sizes d={d}")
    if d < 20:
        run_scan_case(G, oracle, 401, d, 3, batch=1, seed=500 + d, name=f"other sizes d={d}, many chunks")


@pytest.mark.parametrize("d,m", [(3, 2), (5, 8), (8, 3), (7, 12), (16, 5), (13, 16), (20, 7), (32, 5), (24, 32), (50, 33), (33, 50), (64, 20), (61, 64), (100, 37),
                                 (128, 50), (65, 128), (20, 100)])
def test_states_of_another_width(G, oracle, d, m):  # noqa: F811
    run_scan_case(G, oracle, 45, d, 8, m=m, batch=2, seed=600 + d, name=f"other widths d={d} m={m}")


# rows and columns of zeros, entries far apart, the very last entry of the array among them
@pytest.mark.parametrize("d", [3, 7, 11, 15, 18, 35, 51, 77, 127])
def test_zeros_and_wide_entries(G, oracle, d):  # noqa: F811
    T = 24
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 700 + d, T, d))
    Z[5, d - 1] = -np.inf
    Z[9, :, d - 1] = -np.inf
    Z[11] += np.float32(60.0)
    Z[12, d // 2] -= np.float32(70.0)
    re, sg, kap, well = with_sensitivity(lambda z: oracle.scan(z, return_kappa=True), [Z], np.float32, nprobe=2)
    for chunk in (24, 5):
        compare(host(G.scan(dev(Z), chunk_len=chunk)), re, sg, kap, name=f"zeros d={d} chunk={chunk}", max_ill_fraction=0.05, well=well)


# (chunks of one sequence, and of neighbouring sequences, share a wave up to 8 rows)
@pytest.mark.parametrize("value", ["large", "small", "nan", "inf"])
@pytest.mark.parametrize("d", [3, 5, 8, 16])
@pytest.mark.parametrize("chunk", [2, 4, 6, 16])
def test_chains_of_a_wave_do_not_meet(G, oracle, d, chunk, value):  # noqa: F811
    """One factor's magnitude, NaN or infinity changes no bit of what comes before it, or of another sequence."""
    T, at = 34, 21
    z = np.stack([oracle.to_goom(si.normal_chain(si.BASE_SEED + 4100 + d + i, T, d)) for i in range(3)])
    b = np.stack([oracle.to_goom(si.normal_f32(si.BASE_SEED + 4200 + i, 3, T * d).reshape(T, d)) for i in range(3)])
    w = z.copy()
    if value in ("large", "small"):
        w.real[1, at] += 1e6 if value == "large" else -1e6
    else:
        w.real[1, at, 1, d - 1] = np.nan if value == "nan" else np.inf
    for run in (lambda x: G.scan(dev(x), chunk_len=chunk), lambda x: G.affine_scan(dev(x), dev(b), chunk_len=chunk)):
        plain, other = host(run(z)), host(run(w))
        for i in range(3):
            t = at if i == 1 else T
            assert np.array_equal(plain[i, :t].view(np.int64), other[i, :t].view(np.int64)), (i, np.argwhere(plain[i, :t] != other[i, :t])[:4])
    plain, other = host(G.reduce(dev(z), chunk_len=chunk)), host(G.reduce(dev(w), chunk_len=chunk))
    assert np.array_equal(plain[[0, 2]], other[[0, 2]])
