"""128 x 128 products that hold every accumulator to the end: E' and outputs against the
CPU oracle at k around one, two and three ring slabs, at the edge of the k-chunks between
which the accumulators are folded, and with accumulators near the INT32 limit."""
import numpy as np
import pytest

import workloads
from gpu_helpers import from_device, to_device

pytestmark = pytest.mark.gpu


def _run(A, B, N, algo, real=False):
    import torch

    import paper_2512_08321_amd as ozc
    from oracle import core

    m, k = A.shape
    n = B.shape[1]
    print(f"held products {m}x{n}x{k} N={N} {algo} real={real}", flush=True)
    h = ozc.Handle(0, num_moduli=N, algo=algo)
    try:
        if real:
            dA, dB = (torch.from_numpy(np.ascontiguousarray(X.T)).cuda() for X in (A, B))
            C = torch.zeros((n, m), dtype=torch.float64, device="cuda")
            ep = torch.zeros((N, n, m), dtype=torch.int8, device="cuda")
            h.inspect(2, "N", "N", m, n, k, dA, m, dB, k, eprime=ep, C=C, ldc=m)
            ref = core.emulate_real(A, B, N)
            got, want = C.cpu().numpy().T, ref["out"]
            assert np.array_equal(ep.cpu().numpy().transpose(0, 2, 1), ref["Ep"].reshape(N, m, n))
        else:
            dA, dB = to_device(A)[0], to_device(B)[0]
            dC, _ = to_device(np.zeros((m, n), dtype=A.dtype))
            ep = torch.zeros((N, 2, n, m), dtype=torch.int8, device="cuda")
            h.inspect(0, "N", "N", m, n, k, dA, m, dB, k, eprime=ep, C=dC, ldc=m)
            ref = core.emulate(A, B, N, "fast", algo)
            got, want = from_device(dC, m, n, m), ref["out"]
            assert np.array_equal(ep.cpu().numpy().transpose(0, 1, 3, 2), ref["Ep"])
        assert np.array_equal(got, want)
    finally:
        torch.cuda.synchronize()
        h.close()


@pytest.mark.parametrize("algo", ["karatsuba", "4m"])
@pytest.mark.parametrize("k", [1, 64, 65, 128, 129, 192, 256, 32768, 32769, 65600])
def test_k_edges(algo, k):
    m, n = (129, 130) if k < 1000 else (5, 3)
    _run(workloads.complex_matrix(m, k, 0.5, 40 + k), workloads.complex_matrix(k, n, 0.5, 41 + k), 14, algo)


@pytest.mark.parametrize("k", [64, 200, 40000])
def test_real(k):
    A = np.asfortranarray(workloads.complex_matrix(131, k, 1.0, 50).real)
    B = np.asfortranarray(workloads.complex_matrix(k, 17, 1.0, 51).real)
    _run(A, B, 13, "karatsuba", real=True)


@pytest.mark.parametrize("algo", ["karatsuba", "4m"])
@pytest.mark.parametrize("k", [32768, 98304])
def test_equal_signs(algo, k):
    """Constant rows: every term of a product has the same sign and size."""
    A = np.full((3, k), 0.7281 - 0.7281j, order="F") * np.array([[1.0], [0.913], [-0.55]])
    B = np.full((k, 2), -0.611 + 0.947j, order="F")
    _run(np.asfortranarray(A), np.asfortranarray(B), 14, algo)
