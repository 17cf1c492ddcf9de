"""Exponents of a batch's scaling scan: every problem bit-identical with its single call, with
long rows (scanned in several parts), short ones and ragged row groups side by side, both
scaling modes, zero rows and non-finite inputs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (17, 5, 64), (130, 33, 4096), (3, 130, 4097), (64, 64, 9001), (15, 16, 2049),
          (200, 129, 63), (1, 257, 20000)]


@pytest.mark.parametrize("single", [False, True])
@pytest.mark.parametrize("mode", ["fast", "accurate"])
def test_batch_equals_single_calls(mode, single):
    import torch

    import paper_2512_08321_amd as ozc

    dt = torch.complex64 if single else torch.complex128
    N = 7 if single else 14
    print(f"batch scan {mode} single={single}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    h = ozc.Handle(0, num_moduli=N, mode=mode)
    try:
        for bad in (False, True):
            probs, wants = [], []
            for i, (m, n, k) in enumerate(SHAPES):
                ta, tb = "NTC"[i % 3], "NCT"[(i // 2) % 3]
                A = torch.randn((k, m) if ta == "N" else (m, k), dtype=dt, device="cuda", generator=g)
                B = torch.randn((n, k) if tb == "N" else (k, n), dtype=dt, device="cuda", generator=g)
                if m > 2 and ta != "N":
                    A[1] = 0
                if bad and i == 4:
                    B.view(-1)[7] = complex(float("inf"), 1.0)
                C = torch.zeros((n, m), dtype=dt, device="cuda")
                want = torch.zeros_like(C)
                h_call = h.cgemm if single else h.zgemm
                h_call(ta, tb, m, n, k, 1.0, A, A.shape[1], B, B.shape[1], 0.0, want, m)
                probs.append(dict(transa=ta, transb=tb, m=m, n=n, k=k, A=A, lda=A.shape[1], B=B,
                                  ldb=B.shape[1], C=C, ldc=m))
                wants.append(want)
            for _ in range(3):  # recorded once, replayed with other work in between
                for p in probs:
                    p["C"].zero_()
                h.gemm_vbatched(probs, single=single)
                assert h.last_info()["nonfinite"] == int(bad)
                for p, want in zip(probs, wants):
                    assert torch.equal(torch.view_as_real(p["C"]).nan_to_num(7.0),
                                       torch.view_as_real(want).nan_to_num(7.0)), (p["m"], p["n"], p["k"])
    finally:
        torch.cuda.synchronize()
        h.close()
