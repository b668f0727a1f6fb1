"""The default H-product schedule by rows and entries per row: long rows take
sixteen lanes of four entries only where there are rows enough for every compute
unit, and 64 lanes elsewhere (host code: this runs without a GPU)."""
import ctypes as C
import os

import pytest

from paper_2606_29692_amd import binding as B

V = B.VQE_SPMV_VEC4


@pytest.mark.parametrize("n,per_row,want", [
    (1, 2, 8), (10, 11, 8), (10, 12, 16), (12, 39, 16), (12, 40, 32), (18, 95, 32),
    (7, 96, 64 | V), (10, 512, 64 | V), (12, 96, 64 | V), (12, 2048, 64 | V),
    (13, 96, 16 | V), (13, 255, 16 | V), (13, 256, 64 | V), (13, 2048, 64 | V),
    (14, 96, 16 | V), (14, 2048, 16 | V), (20, 200, 16 | V)])
def test_default_schedule(n, per_row, want):
    if not os.path.exists(B.LIB_PATH):
        pytest.skip("libadaptvqe.so is not built")
    H = B.vqe_csr()
    H.n_qubits, H.dim, H.nnz, H.dtype = n, 1 << n, per_row << n, B.VQE_C128
    assert B.lib().vqe_default_schedule(C.byref(H)) == want
