"""Products cut along k (single calls whose tiles leave CUs idle): bit-identical to the
whole products, which ozc_inspect runs, and to a call on a workspace without room for
the parts' E' planes; and one call against the CPU oracle."""
import numpy as np
import pytest

import workloads
from gpu_helpers import from_device, to_device

pytestmark = pytest.mark.gpu
KIND = {"z": 0, "c": 1, "d": 2, "s": 3}


@pytest.mark.parametrize("t,m,n,k,N,mode,algo", [
    ("z", 384, 320, 20000, 14, "fast", "karatsuba"),
    ("z", 5, 3, 70001, 24, "fast", "karatsuba"),
    ("z", 130, 70, 9000, 2, "accurate", "4m"),
    ("c", 100, 260, 8200, 8, "fast", "4m"),
    ("d", 300, 200, 30000, 14, "fast", "karatsuba"),
    ("s", 1, 1, 131072, 6, "accurate", "karatsuba"),
    ("z", 2048, 2048, 2048, 13, "fast", "karatsuba"),   # 256 x 256 tiles, last moduli in parts
    ("c", 1024, 1100, 16384, 6, "fast", "4m"),
    ("d", 1030, 1024, 20000, 5, "accurate", "karatsuba")])
def test_parts_equal_whole(t, m, n, k, N, mode, algo):
    import torch

    import paper_2512_08321_amd as ozc

    dt = {"z": torch.complex128, "c": torch.complex64, "d": torch.float64, "s": torch.float32}[t]
    print(f"k split {t} {m}x{n}x{k} N={N} {mode} {algo}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    A = torch.randn((k, m), dtype=dt, device="cuda", generator=g)
    B = torch.randn((n, k), dtype=dt, device="cuda", generator=g)
    whole, split, tight = (torch.zeros((n, m), dtype=dt, device="cuda") for _ in range(3))
    h = ozc.Handle(0, num_moduli=N, mode=mode, algo=algo)
    try:
        h.inspect(KIND[t], "N", "N", m, n, k, A, m, B, k, C=whole, ldc=m)
        need = h.last_info()["workspace"]
        call = getattr(h, t + "gemm")
        call("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, split, m)
        assert h.last_info()["workspace"] > need  # the case is one that is split
        buf = torch.empty(need, dtype=torch.uint8, device="cuda")
        h.set_workspace(buf, need)
        call("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, tight, m)
        assert h.last_info()["workspace"] == need
        assert torch.equal(whole, split) and torch.equal(whole, tight)
    finally:
        torch.cuda.synchronize()
        h.close()


def test_against_oracle():
    import torch

    import paper_2512_08321_amd as ozc
    from oracle import core

    m, n, k, N = 6, 4, 33000, 14
    A = workloads.complex_matrix(m, k, 1.0, 61)
    B = workloads.complex_matrix(k, n, 1.0, 62)
    C = workloads.complex_matrix(m, n, 1.0, 63)
    h = ozc.Handle(0, num_moduli=N)
    try:
        (dA, _), (dB, _), (dC, _) = to_device(A), to_device(B), to_device(C)
        h.zgemm("N", "N", m, n, k, 0.5 - 1j, dA, m, dB, k, 1.5 + 1j, dC, m)
        got = from_device(dC, m, n, m)
    finally:
        torch.cuda.synchronize()
        h.close()
    assert np.array_equal(got, core.emulate(A, B, N, alpha=0.5 - 1j, beta=1.5 + 1j, C=C)["out"])
