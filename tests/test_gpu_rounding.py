"""Rounding of the reconstructed integers against the CPU oracle: products that are ties,
next to ties, far apart in their high and low parts, or nearly cancel, for every chunk
count of the reconstruction and every element kind."""
import numpy as np
import pytest

from gpu_helpers import from_device, to_device

pytestmark = pytest.mark.gpu


def _operands():
    """Rows whose products with the columns are chosen integers: [hi, lo, 0, 0] . [2^30, 1, ..]."""
    targets = [1, 3, 2**53 + 1, 2**54 + 2, 2**54 + 6, 2**54 + 3, 2**60 + 2**7, 2**60 + 2**7 + 1,
               2**60 + 3 * 2**7, 2**60 + 2**7 - 1, 2**80 + 2**27, 2**80 + 2**27 + 1, 2**80 + 2**27 - 1,
               2**80 + 3 * 2**27, 2**77 + 1, 2**76, 2**75 - 1, 2**38, 2**38 - 1, 2**79 + 2**26 + 2**20]
    rows = [[t >> 30, t & (2**30 - 1), 0, 0] for t in targets]
    rows += [[2**50, 1, -(2**50), 0], [2**50, 3, -(2**50) + 1, 0], [2**45 + 7, 0, -(2**45) - 7, 0],
             [2**50, -1, -(2**50), 0], [2**50 - 1, 2**29, -(2**50) + 2, 5]]
    A = np.array(rows, dtype=float)
    A = np.concatenate([A, -A])
    B = np.array([[2.0**30, 1.0, 2.0**30, 0.0], [2.0**30, 1.0, 2.0**30, 1.0], [2.0**30, -1.0, 2.0**30, 0.5]]).T
    return np.asfortranarray(A), np.asfortranarray(B)


@pytest.mark.parametrize("N", [3, 4, 6, 9, 10, 14, 15, 17, 19, 20, 22, 24])
@pytest.mark.parametrize("mode", ["fast", "accurate"])
def test_rounding(N, mode):
    import torch

    import paper_2512_08321_amd as ozc
    from oracle import core

    A, B = _operands()
    m, k = A.shape
    n = B.shape[1]
    h = ozc.Handle(0, num_moduli=N, mode=mode)
    try:
        for real in (False, True):
            print(f"rounding N={N} {mode} real={real}", flush=True)
            if real:
                a, b = A, B
                dA, dB = (torch.from_numpy(np.ascontiguousarray(x.T)).cuda() for x in (a, b))
                dC = torch.zeros((n, m), dtype=torch.float64, device="cuda")
                h.dgemm("N", "N", m, n, k, 1.0, dA, m, dB, k, 0.0, dC, m)
                got = dC.cpu().numpy().T
                want = core.emulate_real(a, b, N, mode)["out"]
            else:
                a, b = A + 1j * A[::-1], B * (1.0 - 0.0j)
                (dA, _), (dB, _), (dC, _) = to_device(np.asfortranarray(a)), to_device(np.asfortranarray(b)), \
                    to_device(np.zeros((m, n), dtype=complex))
                h.zgemm("N", "N", m, n, k, 1.0, dA, m, dB, k, 0.0, dC, m)
                got = from_device(dC, m, n, m)
                want = core.emulate(a, b, N, mode)["out"]
            assert np.array_equal(got, want)
            same_sign = np.signbit(got.real) == np.signbit(want.real)
            assert same_sign.all()
    finally:
        torch.cuda.synchronize()
        h.close()
