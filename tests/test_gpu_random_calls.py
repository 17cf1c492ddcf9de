"""Plain calls at the seeded configurations of the intermediates' random test, against the
CPU oracle: ozc_inspect takes separate scan and split launches, 128 x 128 tiles and, with
raw products asked for, kernels of their own, so calls without it are checked here.  Real
types, general alpha and beta, and longer inner dimensions among them."""
import numpy as np
import pytest

import workloads
from gpu_helpers import from_device, stored, to_device
from test_gpu_parity import _gemm_call, _random_case, _same, handle, orc  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("i", range(200))
def test_complex(handle, orc, i):  # noqa: F811
    m, n, k, single, N, mode, algo, ta, tb, phi, (pa, pb) = _random_case(i)
    rng = np.random.default_rng(17000 + i)
    if i % 4 == 0:  # small outputs, k past the limit of the one-launch preparation and a part
        m, n, k = 1 + m % 40, 1 + n % 40, 513 + int(rng.integers(0, 5000))
    dt = np.complex64 if single else np.complex128
    A = workloads.complex_matrix(m, k, phi, 8000 + 2 * i, dtype=dt)
    B = workloads.complex_matrix(k, n, phi, 8001 + 2 * i, dtype=dt)
    C = workloads.complex_matrix(m, n, 1.0, 9000 + i, dtype=dt)
    if i % 10 == 1:
        A[m // 2, k // 3] = complex(np.nan, 1.0)
    if i % 10 == 2:
        B[k // 2, n // 3] = complex(0.0, -np.inf)
    alpha, beta = [(1.0, 0.0), (0.5 - 2.0j, 0.0), (1.0, 1.0), (-0.75j, 1.25 + 0.5j)][i % 4]
    print(f"call {i}: {m}x{n}x{k} N={N} {mode} {algo} {ta}{tb} single={single}", flush=True)
    handle.set_config(N, mode, algo)
    (dA, lda), (dB, ldb) = (to_device(S, S.shape[0] + p) for S, p in ((stored(A, ta), pa), (stored(B, tb), pb)))
    dC, ldc = to_device(C, m + 2)
    fn = handle.cgemm if single else handle.zgemm
    fn(ta, tb, m, n, k, alpha, dA, lda, dB, ldb, beta, dC, ldc)
    flag = handle.last_info()["nonfinite"]
    ref = orc.emulate(A, B, N, mode, algo, alpha=alpha, beta=beta, C=C, single=single)
    assert _same(from_device(dC, m, n, ldc), ref["out"])
    assert flag == int(i % 10 in (1, 2))


@pytest.mark.parametrize("i", range(60))
def test_real(handle, orc, i):  # noqa: F811
    import torch

    m, n, k, single, N, mode, _, ta, tb, phi, _ = _random_case(500 + i)
    if i % 4 == 0:
        m, n, k = 1 + m % 40, 1 + n % 40, 513 + 83 * i
    dt = np.float32 if single else np.float64
    A, B, C = (np.asfortranarray(workloads.complex_matrix(r, c, p, 9500 + 3 * i + j).real.astype(dt))
               for j, (r, c, p) in enumerate(((m, k, phi), (k, n, phi), (m, n, 1.0))))
    alpha, beta = [(1.0, 0.0), (-0.75, 1.25)][i % 2]
    print(f"real call {i}: {m}x{n}x{k} N={N} {mode} {ta}{tb} single={single}", flush=True)
    handle.set_config(N, mode, "karatsuba")
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x.T)).cuda()
    dA, dB, dC = dev(A if ta == "N" else A.T), dev(B if tb == "N" else B.T), dev(C)
    fn = handle.sgemm if single else handle.dgemm
    fn(ta, tb, m, n, k, alpha, dA, dA.shape[1], dB, dB.shape[1], beta, dC, m)
    ref = orc.emulate_real(A, B, N, mode, alpha=alpha, beta=beta, C=C, single=single)
    assert _same(dC.cpu().numpy().T, ref["out"])


@pytest.mark.parametrize("algo", ["karatsuba", "4m"])
def test_row_padding_left_from_an_earlier_call(handle, orc, algo):  # noqa: F811
    """As the intermediates' test of that name, with plain calls second and third."""
    A = workloads.complex_matrix(600, 300, 4.0, 901)
    B = workloads.complex_matrix(300, 500, 4.0, 902)
    _gemm_call(handle, A, B, np.zeros((600, 500)), 1.0, 0.0, 20, "fast", algo)
    for m, n, k in ((131, 77, 190), (70, 200, 700)):
        A = workloads.complex_matrix(m, k, 0.5, 903)
        B = workloads.complex_matrix(k, n, 0.5, 904)
        got = _gemm_call(handle, A, B, np.zeros((m, n)), 1.0, 0.0, 14, "fast", algo)
        assert _same(got, orc.emulate(A, B, 14, "fast", algo)["out"])


NEARLY_FULL = ("z", 256, 256, 448, 14, "4m")  # 224 blocks of 64 x 64, four products


def test_64_tiles_nearly_as_many_as_cus():
    from test_gpu_64_tiles import test_equal_to_128_tiles as compare

    compare(*NEARLY_FULL)
