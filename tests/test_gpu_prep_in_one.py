"""Short rows, scanned and split by one launch: outputs bit-identical with the separate scan
and split (which ozc_inspect runs), around the k-slabs and the largest k, with 4 and 16
rows per block, for every element kind and memory order; rows next to a threshold of the
exponent rule, zero rows, and non-finite inputs with their flag."""
import numpy as np
import pytest

from test_gpu_row_scan import _threshold_rows

pytestmark = pytest.mark.gpu
KIND = {"z": 0, "c": 1, "d": 2, "s": 3}


def _check(t, m, n, k, ta, tb, N, algo="karatsuba", edit=None):
    import torch

    import paper_2512_08321_amd as ozc

    print(f"prep in one {t} {m}x{n}x{k} {ta}{tb} N={N} {algo}", flush=True)
    dt = {"z": torch.complex128, "c": torch.complex64, "d": torch.float64, "s": torch.float32}[t]
    g = torch.Generator(device="cuda").manual_seed(m * 7 + k)
    A = torch.randn((k, m + 1) if ta == "N" else (m, k + 1), dtype=dt, device="cuda", generator=g)
    B = torch.randn((n, k + 2) if tb == "N" else (k, n + 2), dtype=dt, device="cuda", generator=g)
    bad = edit(A, B) if edit else 0
    got, want = (torch.zeros((n, m), dtype=dt, device="cuda") for _ in range(2))
    h = ozc.Handle(0, num_moduli=N, algo=algo)
    try:
        h.inspect(KIND[t], ta, tb, m, n, k, A, A.shape[1], B, B.shape[1], C=want, ldc=m)
        assert h.last_info()["nonfinite"] == bad
        getattr(h, t + "gemm")(ta, tb, m, n, k, 1.0, A, A.shape[1], B, B.shape[1], 0.0, got, m)
        assert h.last_info()["nonfinite"] == bad
    finally:
        torch.cuda.synchronize()
        h.close()
    view = torch.view_as_real if dt.is_complex else (lambda x: x)
    assert torch.equal(view(got).nan_to_num(7.0), view(want).nan_to_num(7.0))


@pytest.mark.parametrize("k", [1, 4, 63, 64, 65, 255, 256, 257, 449, 511, 512, 513])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "C")])
def test_k(k, ta, tb):
    _check("z", 131, 66, k, ta, tb, 14)


@pytest.mark.parametrize("t", "zcds")
@pytest.mark.parametrize("m,n", [(1, 1), (5, 3), (4000, 95), (4000, 96), (33, 5000)])
def test_kinds_and_row_groups(t, m, n):
    for k, N, algo in ((100, 6, "4m"), (500, 17, "karatsuba")):
        _check(t, m, n, k, "C" if t in "zc" else "T", "N", N, algo)


@pytest.mark.parametrize("k", [3, 257, 512])
def test_threshold_rows(k):
    import torch

    from oracle import core

    P = int(core.constants(14)["P"])
    mag = torch.from_numpy(_threshold_rows(56, k, 2 * k, P)).cuda()

    def edit(A, B):  # A stored with rows contiguous in k
        A[:, :k] = mag * (1.0 + 1.0j)
        A[7] = 0
        return 0

    _check("z", 56, 40, k, "T", "N", 14, edit=edit)


@pytest.mark.parametrize("where", ["A", "B"])
def test_nonfinite(where):
    def edit(A, B):
        (A if where == "A" else B)[4, 9] = complex(np.nan, 0.0) if where == "A" else complex(0.0, -np.inf)
        return 1

    _check("z", 70, 130, 200, "T", "N", 12, edit=edit)
