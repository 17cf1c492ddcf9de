"""Fast-mode exponents of the one-read scan against the CPU oracle: ragged rows and k
around the block's 16 rows x 64 lanes x 8 loads, rows scanned in one and in several
parts, both memory orders and every element kind; rows whose sum of squares lies next
to a threshold of the rule (only the exact integer sum decides those), rows outside the
range of FP64 squares, zero rows and rows holding inf or NaN."""
from math import isqrt

import numpy as np
import pytest

import workloads
from gpu_helpers import oracle_exp, stored, to_device

pytestmark = pytest.mark.gpu
N = 14


@pytest.fixture(scope="module")
def handle():
    import torch

    import paper_2512_08321_amd as ozc

    h = ozc.Handle(0, num_moduli=N)
    yield h
    torch.cuda.synchronize()
    h.close()


def _threshold_rows(rows, k, nreal, P):
    """Rows of constant magnitude y 2^(e - 20), so sigma = nreal y^2 (ceil(y)^2 off the
    integers), with nreal y^2 within a few y of a threshold (P - 1) 2^37 / 4^t."""
    t = 0
    while not (1 << 20) <= isqrt(((P - 1) << 37 >> (2 * t)) // nreal) < (1 << 21) - 8:
        t += 1
    y0 = isqrt(((P - 1) << 37 >> (2 * t)) // nreal)
    steps = [0.0, 1.0, -1.0, 0.5, -0.5, 2.0, -2.0, 5.0]
    exps = [0, 3, -60, 470, -470, 449, -449]
    mag = np.array([np.ldexp(y0 + steps[r % 8], exps[r % 7] - 20) for r in range(rows)])
    return np.repeat(mag[:, None], k, axis=1)


def _exponents(h, kind, A, B, ta, tb):
    import torch

    m, k = A.shape
    n = B.shape[1]
    print(f"row scan kind={kind} m,n,k={m},{n},{k} {ta}{tb}", flush=True)
    dt = {0: np.complex128, 1: np.complex64, 2: np.float64, 3: np.float32}[kind]
    bufs = []
    for X, op in ((A, ta), (B, tb)):
        S = stored(X, op)
        if kind < 2:
            bufs.append(to_device(np.asfortranarray(S.astype(dt)), S.shape[0] + 1))
        else:
            bufs.append((torch.from_numpy(np.ascontiguousarray(S.real.T.astype(dt))).cuda(), S.shape[0]))
    mu = torch.zeros(m, dtype=torch.int16, device="cuda")
    nu = torch.zeros(n, dtype=torch.int16, device="cuda")
    h.set_config(N)
    h.inspect(kind, ta, tb, m, n, k, bufs[0][0], bufs[0][1], bufs[1][0], bufs[1][1], mu, nu,
              ldc=m)
    return mu.cpu().numpy(), nu.cpu().numpy()


def _check(h, kind, A, B, ta="N", tb="N"):
    from oracle import core

    got = _exponents(h, kind, A, B, ta, tb)
    flag = h.last_info()["nonfinite"]
    for g, (re, im), what in zip(got, (core.rows_of_A(A), core.rows_of_B(B)), ("mu", "nu")):
        e, f = core.fast_exponents(re, im, N)[:2]
        assert np.array_equal(g, oracle_exp(e, f)), what
    assert flag == int(not (np.isfinite(A).all() and np.isfinite(B).all()))


@pytest.mark.parametrize("k", [1, 63, 65, 511, 513, 4096, 4097, 9001])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "T")])
def test_ragged(handle, k, ta, tb):
    m, n = (17, 130) if k < 4096 else (33, 15)
    A = workloads.complex_matrix(m, k, 2.0, 700 + k)
    B = workloads.complex_matrix(k, n, 0.5, 800 + k)
    A[3, :] = 0.0
    B[:, 1] = 0.0
    _check(handle, 0, A, B, ta, tb)
    A[5, k // 2] = complex(np.inf, 1.0)
    B[k - 1, 2] = complex(0.0, np.nan)
    _check(handle, 0, A, B, ta, tb)


@pytest.mark.parametrize("kind", [1, 2, 3])
def test_kinds(handle, kind):
    for k in (70, 5000):
        A = workloads.complex_matrix(40, k, 1.0, 900)
        B = workloads.complex_matrix(k, 19, 1.0, 901)
        if kind >= 2:
            A, B = A.real + 0j, B.real + 0j
        if kind in (1, 3):
            A, B = A.astype(np.complex64).astype(complex), B.astype(np.complex64).astype(complex)
        if kind < 2:
            _check(handle, kind, A, B, "C", "N")
        else:
            from oracle import core

            got = _exponents(handle, kind, A, B, "T", "N")
            # a real row has k reals: same exponents as the complex rule on zero imaginary parts
            for g, (re, im) in zip(got, (core.rows_of_A(A), core.rows_of_B(B))):
                e, f = core.fast_exponents(re, np.zeros_like(im), N)[:2]
                assert np.array_equal(g, oracle_exp(e, f))


@pytest.mark.parametrize("k", [5, 257, 6000])
@pytest.mark.parametrize("ta,tb", [("N", "T"), ("T", "N")])
def test_rows_next_to_a_threshold(handle, k, ta, tb):
    from oracle import core

    P = int(core.constants(N)["P"])
    mag = _threshold_rows(56, k, 2 * k, P)
    A = mag * (1.0 + 1.0j)
    B = np.asfortranarray((mag[:40] * (1.0 - 1.0j)).T)
    _check(handle, 0, np.asfortranarray(A), B, ta, tb)
