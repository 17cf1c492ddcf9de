"""Memory of rows scanned in several parts (the library's own sizes, which need no GPU):
it goes where the residues will be written, and fits at the fewest moduli and planes."""
import ctypes

import paper_2512_08321_amd as ozc


def test_parts_fit_the_residues():
    L = ctypes.CDLL(ozc.library_path)
    parts, scratch = L._ZN3ozc14row_scan_partsEll, L._ZN3ozc16row_scan_scratchEll
    for f in (parts, scratch):
        f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_int64] * 2
    seen = set()
    for k in [1, 64, 4096, 4097, 4160, 5000, 6145, 8191, 8193, 20000, 65537, 100000, ozc.MAX_K]:
        for groups in (0, 16, 17, 40, 100, 300, 511, 512, 5000):
            p = parts(k, groups)
            seen.add(p > 1)
            assert p == 1 if k <= 4096 or groups >= 512 else 1 <= p <= (k + 2047) // 2048
            chunk = (k + p - 1) // p
            assert (p - 1) * chunk < k <= p * chunk and (p == 1 or chunk >= 1024)  # no empty part
            for rows in (128, 256, 8192):
                need = scratch(rows, p)
                # [p][rows] maxima and sums of squares, [rows] sums, a counter per 16 rows
                assert need == (0 if p == 1 else rows * (16 * p + 8) + rows // 4)
                assert need <= ozc.MIN_MODULI * rows * ((k + 63) // 64 * 64)
    assert seen == {False, True}
