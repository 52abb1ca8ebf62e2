"""The rule that cuts 2D problems into segments, called in the library without a
GPU: a caller's height stands wherever its tiles occupy the GPU's workgroup
slots, the height a handle starts with may be shortened below two rounds of
them, and problems that leave slots empty are cut."""
import ctypes as C

import pytest

from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

# workgroups per CU by registers and LDS: F64, F32, F32_ACC64, F32_KAHAN
SLOTS = {(0, 2): (3, 5, 5, 5), (0, 3): (2, 4, 4, 4), (1, 2): (1, 3, 3, 3), (1, 3): (1, 2, 2, 2)}


def _split(specs, cfg, cap):
    f = hw.lib()._ZN5hweno10split_rowsEPK13hweno_problemiRK12hweno_configi
    f.restype, f.argtypes = C.c_int, [C.c_void_p, C.c_int, C.c_void_p, C.c_int]
    probs = (hw.hweno_problem * len(specs))(*[hw.problem(s) for s in specs])
    return f(C.addressof(probs), len(specs), C.addressof(cfg), cap)


def _tiles(specs, rows):
    return sum(-(-s.nx // 60) * -(-s.ny // rows) for s in specs)


@pytest.mark.parametrize("charwise", [0, 1])
@pytest.mark.parametrize("q", [2, 3])
@pytest.mark.parametrize("prec", [hw.F64, hw.F32, hw.F32_ACC64, hw.F32_KAHAN])
def test_a_callers_height_stands_where_it_fills_the_gpu(prec, q, charwise):
    cfg = hw.default_config(2, precision=prec, gauss_q=q, characteristic=charwise)
    slots = 256 * SLOTS[charwise, q][prec]
    for n in ((2048, 2048), (1500, 1500), (4096, 300), (256, 256), (97, 1031)):
        one = W.Spec(dim=2, flux=W.EULER, nx=n[0], ny=n[1], t_end=1.0)
        for specs in ([one], [one] * 24):
            for cap in (8, 13, 16, 24, 31, 33, 36, 48, 57, 64, 128, 1024):
                rows = _split(specs, cfg, cap)
                if _tiles(specs, cap) >= slots:
                    assert rows == cap, (n, len(specs), cap, rows)
                else:
                    assert 2 <= rows <= cap, (n, len(specs), cap, rows)
                    assert _tiles(specs, rows) >= _tiles(specs, cap)
            rows = _split(specs, cfg, 32)
            if _tiles(specs, 32) >= 2 * slots:
                assert rows == 32
            else:
                assert 2 <= rows <= 32


def test_small_problems_are_cut():
    cfg = hw.default_config(2, precision=hw.F64, gauss_q=3)
    spec = W.Spec(dim=2, flux=W.EULER, nx=256, ny=256, t_end=1.0)
    for cap in (16, 32, 64):
        assert _tiles([spec], _split([spec], cfg, cap)) >= 256
