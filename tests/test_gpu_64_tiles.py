"""Products on 64 x 64 tiles (single calls that leave CUs idle): bit-identical to the
128 x 128 tiles, which ozc_inspect runs."""
import pytest

pytestmark = pytest.mark.gpu
KIND = {"z": 0, "c": 1, "d": 2, "s": 3}


@pytest.mark.parametrize("t,m,n,k,N,algo", [
    ("z", 1, 1, 1, 14, "karatsuba"),
    ("z", 64, 64, 64, 14, "karatsuba"),
    ("z", 63, 65, 65, 20, "4m"),
    ("z", 129, 1, 200, 3, "karatsuba"),
    ("z", 256, 256, 512, 14, "4m"),        # as many blocks as it has CUs, but for 32
    ("c", 333, 777, 555, 8, "karatsuba"),  # more blocks than CUs
    ("c", 2, 1600, 128, 4, "4m"),
    ("d", 65, 64, 1000, 14, "karatsuba"),
    ("s", 300, 190, 129, 6, "karatsuba")])
def test_equal_to_128_tiles(t, m, n, k, N, algo):
    import torch

    import paper_2512_08321_amd as ozc

    dt = {"z": torch.complex128, "c": torch.complex64, "d": torch.float64, "s": torch.float32}[t]
    print(f"64 x 64 tiles {t} {m}x{n}x{k} N={N} {algo}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    A = torch.randn((k, m), dtype=dt, device="cuda", generator=g)
    B = torch.randn((n, k), dtype=dt, device="cuda", generator=g)
    large, small = (torch.zeros((n, m), dtype=dt, device="cuda") for _ in range(2))
    h = ozc.Handle(0, num_moduli=N, algo=algo)
    try:
        h.inspect(KIND[t], "N", "N", m, n, k, A, m, B, k, C=large, ldc=m)
        getattr(h, t + "gemm")("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, small, m)
        assert torch.equal(large, small)
    finally:
        torch.cuda.synchronize()
        h.close()
