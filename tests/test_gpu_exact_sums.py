"""The scaling scan where many or all rows need their exact integer sums (magnitudes beyond
the range of FP64 squares, rows next to a threshold): exponents against the CPU oracle
around the count at which a block takes its rows together, in one and in several parts, in
both memory orders; batches against single calls; and the time of such a call, which is one
more read of the operands and not a serial walk over them."""
import numpy as np
import pytest

import workloads
from test_gpu_row_scan import N, _check, _threshold_rows, handle  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [3, 64, 1000, 4500, 9001, 20000])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "T")])
def test_open_rows_in_a_group(handle, k, ta, tb):  # noqa: F811
    # groups of 16 rows with 0 .. 16 of them beyond the range, large or small
    m, n = (16 * 17, 21) if k < 9000 else (70, 40)
    A = workloads.complex_matrix(m, k, 1.0, 300 + k)
    B = workloads.complex_matrix(k, n, 2.0, 301 + k)
    for r in range(m):
        g, i = divmod(r, 16)
        count = g if m > 70 else [4, 5, 16, 1, 9][g]
        if (7 * i) % 16 < count:
            A[r] *= 2.0 ** (500 if (r + g) % 2 else -500)
    B *= 2.0 ** -900
    B[:, 3] = 0.0
    A[1, k - 1] = np.nan
    _check(handle, 0, np.asfortranarray(A), np.asfortranarray(B), ta, tb)


@pytest.mark.parametrize("kind", [1, 2, 3])
@pytest.mark.parametrize("k", [700, 6100])
def test_kinds_next_to_a_threshold(handle, kind, k):  # noqa: F811
    from oracle import core
    from gpu_helpers import oracle_exp
    from test_gpu_row_scan import _exponents

    P = int(core.constants(N)["P"])
    nreal = 2 * k if kind == 1 else k
    mag = _threshold_rows(40, k, nreal, P)
    if kind in (1, 3):  # within float's range: 24 bits hold y and its halves
        mag = np.ldexp(np.frexp(mag)[0], np.arange(40)[:, None] % 50 - 20)
    f = 1.0 + 1.0j if kind == 1 else 1.0 + 0.0j
    A, B = np.asfortranarray(mag * f), np.asfortranarray((mag[:23] * f).T)
    for ta, tb in (("N", "N"), ("T", "T")):
        got = _exponents(handle, kind, A, B, ta, tb)
        for g, (re, im) in zip(got, (core.rows_of_A(A), core.rows_of_B(B))):
            e, fl = core.fast_exponents(re, im if kind == 1 else np.zeros_like(im), N)[:2]
            assert np.array_equal(g, oracle_exp(e, fl))


def test_batch_equals_single_calls(handle):  # noqa: F811
    import torch

    g = torch.Generator(device="cuda").manual_seed(8)
    rand = lambda *s: torch.randn(s, dtype=torch.complex128, device="cuda", generator=g)
    probs, want = [], []
    for i, (m, n, k) in enumerate([(33, 17, 5000), (130, 64, 4096), (5, 300, 12000), (64, 64, 64), (40, 9, 30000)]):
        A, B = rand(k, m), rand(n, k)
        if i != 3:
            A *= 2.0 ** -520
            B[: n // 2] *= 2.0 ** 470
        C, D = (torch.zeros((n, m), dtype=torch.complex128, device="cuda") for _ in range(2))
        probs.append({"transa": "N", "transb": "N", "m": m, "n": n, "k": k, "alpha": 1.0, "A": A, "lda": m,
                      "B": B, "ldb": k, "beta": 0.0, "C": C, "ldc": m})
        handle.zgemm("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, D, m)
        want.append(D)
    for _ in range(3):
        handle.gemm_vbatched(probs)
        assert all(torch.equal(p["C"], w) for p, w in zip(probs, want))
        for p in probs:
            p["C"].zero_()


@pytest.mark.parametrize("t,m,n,k,ta", [("z", 384, 320, 40000, "N"), ("d", 8000, 64, 9000, "N"),
                                        ("z", 2048, 2048, 2048, "T")])
def test_time_beyond_the_range_of_squares(t, m, n, k, ta):
    """At most twice the call within the range (before exact sums had the whole chip: 2.9
    times for the first two)."""
    import torch

    import paper_2512_08321_amd as ozc

    dt = {"z": torch.complex128, "d": torch.float64}[t]
    h = ozc.Handle(0, num_moduli=N)
    try:
        A, B = torch.randn((k * m,), dtype=dt, device="cuda"), torch.randn((n * k,), dtype=dt, device="cuda")
        C = torch.zeros((n, m), dtype=dt, device="cuda")
        us = []
        for scale in (1.0, 2.0 ** -500):
            A.mul_(scale)
            B.mul_(scale)
            best = float("inf")
            for _ in range(6):
                e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                e0.record()
                for _ in range(4):
                    getattr(h, t + "gemm")(ta, "N", m, n, k, 1.0, A, m if ta == "N" else k, B, k, 0.0, C, m)
                e1.record()
                e1.synchronize()
                best = min(best, e0.elapsed_time(e1) * 250.0)
            us.append(best)
        print(f"{t} {m}x{n}x{k}: {us[0]:.0f} us, beyond the range {us[1]:.0f} us", flush=True)
        assert us[1] < 2.0 * us[0]
    finally:
        torch.cuda.synchronize()
        h.close()
