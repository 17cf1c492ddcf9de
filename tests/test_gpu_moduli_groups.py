"""Batched products whose blocks take several moduli of a tile in a row: each starts on the
LDS ring that the one before has just read, at every buffer the last slab can stand in.
Bit-identical to single calls and to one modulus at a time."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo", ["karatsuba", "4m"])
@pytest.mark.parametrize("single", [False, True])
def test_groups_equal_single_calls(algo, single):
    import torch

    import paper_2512_08321_amd as ozc

    N = 9 if single else 14
    dt = torch.complex64 if single else torch.complex128
    g = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *s: torch.randn(s, dtype=dt, device="cuda", generator=g)
    # 1 .. 8 slabs of 64: three or four products of them end in each buffer of the ring;
    # tiles of 128, and one of 256
    shapes = [(130, 129, 64 * s - 7 * (s % 3)) for s in range(1, 9)] + [(40, 300, 1000), (300, 270, 100)]
    h = ozc.Handle(0, num_moduli=N, algo=algo)
    try:
        ops = [(m, n, k, rand(k, m), rand(n, k)) for m, n, k in shapes]
        want = []
        for m, n, k, A, B in ops:
            C = torch.zeros((n, m), dtype=dt, device="cuda")
            (h.cgemm if single else h.zgemm)("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, C, m)
            want.append(C)
        for group in (1, 2, 3, N, N + 5):
            print(f"moduli group {group} {algo} single={single}", flush=True)
            h.set_batch_policy(tile_threshold=256, moduli_group=group, use_graph=group % 2 == 0)
            out = [torch.full_like(C, float("nan")) for C in want]
            for _ in range(3):
                h.gemm_vbatched([{"transa": "N", "transb": "N", "m": m, "n": n, "k": k, "alpha": 1.0, "A": A,
                                  "lda": m, "B": B, "ldb": k, "beta": 0.0, "C": C, "ldc": m}
                                 for (m, n, k, A, B), C in zip(ops, out)], single=single)
                assert all(torch.equal(a, b) for a, b in zip(want, out))
    finally:
        torch.cuda.synchronize()
        h.close()
