"""Chunk products [A* | b*] of the recurrence at d = 64: the bias column, sixteen rows to a wave on powers of two of their own.  Chunks at and
beside the column's renormalisation (every four steps), and rows of one wave that are zero, or far above or below another's."""
import numpy as np
import pytest

import synthetic_inputs as si
from test_gpu_parity import G, compare, dev, host, say, with_sensitivity  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [1, 2, 3, 4, 5, 8, 21])
def test_rows_of_one_wave_unlike_another(G, oracle, chunk):  # noqa: F811
    batch, T, d = 9, 43, 64
    A, b = si.recurrence_inputs(si.BASE_SEED + 1200, batch, T, d)
    Az, bz = oracle.to_goom(A), oracle.to_goom(b)
    zero = np.complex64(complex(-np.inf, 0.0))
    Az[0, :, 16:32] = zero     # a wave's rows without terms: the bias alone
    bz[1, :, 32:48] = zero     # ... without biases
    Az[2, :, 48:] = zero       # ... without either
    bz[2, :, 48:] = zero
    bz[3, :, :16] += 300       # biases e^300 above and below the others'
    bz[3, :, 16:32] -= 300
    Az[4] += 40                # log-magnitudes reach 1700
    bz[5] = zero               # nothing but zeros until h0
    bz[6, :9] = zero           # the column starts late
    Az[7, 10] = zero           # a zero matrix: the state restarts from the bias
    Az[7, 11, 20:30] = zero
    Az[8, :, :16, 16:] = zero  # a block that keeps to itself and grows by e^20 a step
    Az[8, :, :16] += 20
    h0 = oracle.to_goom(si.normal_f32(si.BASE_SEED + 1201, 9, batch * d).reshape(batch, d))
    say(f"augmented chunk products, chunk={chunk}")
    fn = lambda a_, b_, h_: oracle.affine_scan(a_, b_, h0=h_, return_kappa=True)
    for start in (None, h0):
        re, sg, kap, well = with_sensitivity(fn, [Az, bz, start], np.float32)
        got = host(G.affine_scan(dev(Az), dev(bz), None if start is None else dev(start), chunk_len=chunk))
        assert np.array_equal(np.isneginf(got[5].real), np.isneginf(re[5]))
        compare(got, re, sg, kap, name=f"chunk{chunk}", max_ill_fraction=0.05, well=well)
