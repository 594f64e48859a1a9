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
