"""bench.py's bytes of the memory-side phases: one read of the operands for the scan, and no
figure where the scan has no launch of its own or shares its phase with the bound product."""
import pytest


@pytest.mark.parametrize("k,mode,scale", [(16384, "fast", True), (513, "fast", True), (512, "fast", False),
                                          (16384, "accurate", False)])
def test_phase_rates(k, mode, scale):
    from bench import phase_rates, scan_reads

    m, n, N = 4096, 2048, 14
    prof = {"calls": 2, "scale_ms": 2.0, "split_ms": 4.0, "crt_ms": 6.0}
    rates = phase_rates(m, n, k, N, False, "karatsuba", mode, prof, scan_reads(k))
    operands = (m + n) * k * 16
    want = {"split": operands * (16 + 3 * N) / 16 / 2e-3, "crt": m * n * (2 * N + 16) / 3e-3}
    if scale:
        want["scale"] = operands / 1e-3
    assert set(rates) == set(want)
    for key, v in want.items():
        assert rates[key] == pytest.approx(v / 1e12, abs=1e-3)
