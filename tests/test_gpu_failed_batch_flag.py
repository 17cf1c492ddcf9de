"""The non-finite flag after a batch that fails before any of its work is enqueued: such a
call met no input, so the flag of the call before it does not stand."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("verify", [False, True])
def test_flag_of_an_earlier_call_is_cleared(verify):
    import torch

    import paper_2512_08321_amd as ozc

    h = ozc.Handle(0, num_moduli=14)
    try:
        A, B, C = (torch.ones((8, 8), dtype=torch.complex128, device="cuda") for _ in range(3))

        def problem(n):
            return [{"transa": "N", "transb": "N", "m": n, "n": n, "k": 8, "alpha": 1.0, "A": A, "lda": n,
                     "B": B, "ldb": 8, "beta": 0.5, "C": C, "ldc": n}]

        h.set_verify(False)
        h.gemm_vbatched(problem(8))
        assert h.last_info()["nonfinite"] == 0
        A[2, 3] = float("nan")
        h.gemm_vbatched(problem(8))
        assert h.last_info()["nonfinite"] == 1
        h.set_verify(verify)
        # 400 000 squared: its workspace (with the check: the copy of C) exceeds the memory
        print(f"failing batch, verify={verify}", flush=True)
        with pytest.raises(ozc.OzcError) as e:
            h.gemm_vbatched(problem(400000))
        assert e.value.status == 3
        assert h.last_info()["nonfinite"] == 0
    finally:
        torch.cuda.synchronize()
        h.close()
