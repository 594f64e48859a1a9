"""The scan's backward walk where matrices and states fill their tiles: no initial state and one, single steps, chunks with a shorter last one."""
import numpy as np
import pytest

from test_gpu_parity import G  # noqa: F401
from test_gpu_scan_adjoint import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ctype", [np.complex64, np.complex128])
@pytest.mark.parametrize("with_init", [False, True])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_full_tiles(G, oracle, d, with_init, ctype):  # noqa: F811
    run(G, oracle, 1, d, d, 2, 0, ctype, with_init)
    run(G, oracle, 9, d, d, 2, 4, ctype, with_init)
