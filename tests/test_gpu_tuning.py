"""What the tuner times: launches that differ.  Register variants only where the
kernel has two, one candidate where workgroups hold whole problems, and segment
heights that the library does not cut to the same segments."""
import pytest

from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W
from test_segment_heights import _split

pytestmark = pytest.mark.gpu


def _candidates(specs, cfg):
    with hw.Handle(specs, cfg) as h:
        return [(c.tile_rows, c.grid_blocks, c.variant) for c in h.tuning_candidates()]


@pytest.mark.parametrize("n", [96, 600, 2048])
@pytest.mark.parametrize("prec,charwise", [(hw.F64, 0), (hw.F32_ACC64, 0), (hw.F32_ACC64, 1)])
def test_2d_candidates_differ(prec, charwise, n):
    spec = W.Spec(dim=2, flux=W.EULER, nx=n, ny=n, t_end=1.0)
    cfg = hw.default_config(2, precision=prec, gauss_q=2, characteristic=charwise)
    cands = _candidates([spec], cfg)
    assert cands[0] == (32, 0, 0)
    assert len(set(cands)) == len(cands)
    variants = {0, 1} if prec != hw.F64 and not charwise else {0}
    assert {v for _, _, v in cands} == variants
    launches = set()
    for rows, grid, v in cands:
        r = rows if grid else _split([spec], cfg, rows)
        tiles = -(-n // 60) * -(-n // r)
        launches.add((-(-n // r), grid if 0 < grid < tiles else 0, v))
    assert len(launches) == len(cands)


def test_1d_candidates_differ():
    small = [W.Spec(dim=1, flux=W.EULER, nx=nx, t_end=1.0) for nx in (50, 416)]
    assert _candidates(small, hw.default_config(1)) == [(32, 0, 0)]
    # 77 waves: every persistent grid would hold them all
    one = [W.Spec(dim=1, flux=W.EULER, nx=4000, t_end=1.0)]
    assert _candidates(one, hw.default_config(1)) == [(32, 0, 0)]
    many = _candidates(one * 200, hw.default_config(1))
    assert many[0] == (32, 0, 0) and len(many) == 4
