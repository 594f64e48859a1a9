"""Chains over factored matrices (the carries of scans, products of groups of chunk products): around the tiles, states of their own width, rings of
factors shorter and longer than the chain, matrices far from 1, columns of zeros, with and without a bias."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, compare, dev, host, run_scan_case, with_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu

BOTH = [np.float32, np.float64]


# chunks of one step: the carries do all the work; 2 .. 8 of them in one chain, 97 and more in groups
@pytest.mark.parametrize("dtype", BOTH)
@pytest.mark.parametrize("d,m,T", [(1, None, 5), (15, None, 3), (16, 3, 8), (17, None, 7), (33, 50, 6), (50, 33, 4), (64, None, 7), (65, 128, 5), (113, None, 3),
                                   (128, 100, 4), (8, None, 100), (16, 16, 131), (31, 9, 112), (63, None, 103), (64, 64, 99)])
def test_carries(G, oracle, d, m, T, dtype):  # noqa: F811
    run_scan_case(G, oracle, T, d, 1, m=m, batch=2, seed=800 + d, dtype=dtype, name=f"carries d={d} m={m}")


# log-magnitudes of thousands, items in units of their own, zero columns and rows: exponents are kept, and zeros stay zeros
@pytest.mark.parametrize("dtype", BOTH)
@pytest.mark.parametrize("d,T", [(16, 9), (32, 120), (64, 9), (128, 7)])
def test_carries_far_from_one(G, oracle, d, T, dtype):  # noqa: F811
    Z = oracle.to_goom(si.normal_chain(si.BASE_SEED + 900 + d, T, d).astype(dtype))
    Z[1] += dtype(3000.0)
    Z[3] -= dtype(9000.0)
    Z[2, :, d - 1] = -np.inf
    Z[T - 2, d // 2] = -np.inf
    comp = np.dtype(dtype).type
    re, sg, kap, well = with_sensitivity(lambda z: oracle.scan(z, return_kappa=True), [Z], comp, nprobe=2)
    compare(host(G.scan(dev(Z), chunk_len=1)), re, sg, kap, name=f"far from one d={d}", max_ill_fraction=0.05, well=well)
    compare(host(G.reduce(dev(Z), chunk_len=1)), re[-1], sg[-1], kap[-1], name=f"far from one d={d}, last", max_ill_fraction=0.08, well=well[-1])


# products of groups of [A | b]: vectors beside the matrices, far below and far above them
@pytest.mark.parametrize("dtype", BOTH)
@pytest.mark.parametrize("d,shift", [(5, 0.0), (16, 40.0), (24, -40.0), (64, 0.0), (100, 700.0)])
def test_products_with_a_vector(G, oracle, d, shift, dtype):  # noqa: F811
    T, batch = 110, 2
    comp = np.dtype(dtype).type
    A = oracle.to_goom((si.normal_f32(si.BASE_SEED + 950 + d, 1, batch * T * d * d).reshape(batch, T, d, d) * 1.05 / np.sqrt(d)).astype(dtype))
    b = oracle.to_goom(si.normal_f32(si.BASE_SEED + 951 + d, 2, batch * T * d).reshape(batch, T, d).astype(dtype))
    b[:, 1::7] += comp(shift)
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 952 + d, 3, batch * d).reshape(batch, d).astype(dtype))
    got = host(G.affine_scan(dev(A), dev(b), dev(h0), chunk_len=1))
    for i in range(batch):
        re, sg, kap, well = with_sensitivity(lambda x, y, z: oracle.affine_scan(x, y, h0=z, return_kappa=True), [A[i], b[i], h0[i]], comp, nprobe=2)
        compare(got[i], re, sg, kap, name=f"with a vector d={d}", max_ill_fraction=0.1, well=well)
