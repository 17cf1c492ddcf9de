"""The Freivalds check's sums at the edges of their chunks and load batches: the ratio it
reports for a product of two moduli (far off, so the check fails), against the same sums in
NumPy.  Float64 sums of 3100 terms at most are off by less than 3100 2^-53, times three for the
products in them: 1e-12 of the absolute sums.  The largest residual is asserted to be 1e-6 of
them or more, so the ratios agree to 1e-6."""
import numpy as np
import pytest

from gpu_helpers import from_device, to_device
import workloads

pytestmark = pytest.mark.gpu


def signs(seed, n):
    mask = (1 << 64) - 1
    out = []
    for i in range(n):
        z = (seed + (i + 1) * 0x9E3779B97F4A7C15) & mask
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & mask
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
        out.append(-1.0 if (z ^ (z >> 31)) & 1 else 1.0)
    return np.array(out)


@pytest.mark.parametrize("ta,tb,m,n,k,beta", [
    ("N", "N", 1, 1, 1, 0.0), ("N", "N", 5, 7, 8, 0.0), ("N", "N", 257, 9, 31, 0.5),
    ("N", "T", 255, 33, 65, 0.0), ("T", "C", 64, 40, 63, 0.5), ("C", "N", 3, 1025, 449, 0.0),
    ("T", "T", 30, 520, 513, 0.0), ("N", "N", 20, 1030, 2047, -2.0)])
def test_ratio(ta, tb, m, n, k, beta):
    import torch

    import paper_2512_08321_amd as ozc

    print(f"check sums {ta}{tb} {m}x{n}x{k} beta {beta}", flush=True)
    op = {"N": lambda x: x, "T": lambda x: x.T, "C": lambda x: x.conj().T}
    A = workloads.complex_matrix(*((m, k) if ta == "N" else (k, m)), 0.5, 71)
    B = workloads.complex_matrix(*((k, n) if tb == "N" else (n, k)), 0.5, 72)
    C = workloads.complex_matrix(m, n, 0.5, 73)
    seed, rel, alpha = 0x5EED, 1e-12, 1.5 - 0.25j
    h = ozc.Handle(0, num_moduli=2)
    try:
        h.set_verify(True, rel=rel, escalate=False, seed=seed)
        (dA, lda), (dB, ldb), (dC, ldc) = to_device(A), to_device(B), to_device(C)
        try:
            h.zgemm(ta, tb, m, n, k, alpha, dA, lda, dB, ldb, beta, dC, ldc)
        except ozc.OzcError:
            pass
        info = h.last_info()
        got = from_device(dC, m, n, ldc)
    finally:
        torch.cuda.synchronize()
        h.close()
    a, b, x = op[ta](A), op[tb](B), signs(seed, n)
    res = np.abs(got @ x - alpha * (a @ (b @ x)) - beta * (C @ x))
    tol = rel * (abs(alpha) * (np.abs(a) @ (np.abs(b) @ np.abs(x))) + abs(beta) * (np.abs(C) @ np.abs(x)))
    assert (res > 2 * tol).all() and (res / tol).max() > 1e6
    assert info["verify_failed_rows"] == m
    assert abs(info["verify_ratio"] - (res / tol).max()) <= 1e-6 * (res / tol).max()
