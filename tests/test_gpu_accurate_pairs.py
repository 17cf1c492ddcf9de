"""Accurate-mode calls whose operands differ in rows and in which direction is contiguous:
the launches that take both operands (magnitudes, exponents), bit for bit against the oracle."""
import numpy as np
import pytest

import workloads
from gpu_helpers import from_device, stored, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb,m,n,k,N", [
    ("N", "N", 1, 300, 1, 14), ("T", "N", 300, 1, 65, 9), ("N", "C", 129, 33, 64, 14),
    ("C", "T", 31, 257, 130, 12), ("T", "T", 64, 5, 63, 20)])
def test_against_oracle(ta, tb, m, n, k, N):
    import torch

    import paper_2512_08321_amd as ozc
    from oracle import core

    print(f"accurate pairs {ta}{tb} {m}x{n}x{k} N={N}", flush=True)
    A = workloads.complex_matrix(m, k, 2.0, 81)
    B = workloads.complex_matrix(k, n, 2.0, 82)
    h = ozc.Handle(0, num_moduli=N, mode="accurate")
    try:
        (dA, lda), (dB, ldb) = to_device(stored(A, ta)), to_device(stored(B, tb))
        dC = torch.empty((n, m), dtype=torch.complex128, device="cuda")
        h.zgemm(ta, tb, m, n, k, 1.0, dA, lda, dB, ldb, 0.0, dC, m)
        got = from_device(dC, m, n, m)
    finally:
        torch.cuda.synchronize()
        h.close()
    assert np.array_equal(got, core.emulate(A, B, N, mode="accurate")["out"])
