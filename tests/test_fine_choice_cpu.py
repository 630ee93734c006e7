"""Tile choice of products near the end of the fine tiles' range: shapes timed on
both kinds of tiles, with the one that was faster.  work_items of a plan of
128 x 128 tiles in one part is their number; 64 x 64 tiles are about four times
as many."""
import pytest

import paper_1902_02104_amd as P


def _tri(n, t):
    k = -(-n // t)
    return k * (k + 1) // 2


@pytest.mark.parametrize("m,n", [(672, 3819), (684, 3914), (744, 3885), (842, 3950), (795, 3918), (432, 3734),
                                 (158, 3240)])
def test_f32_on_128_tiles(m, n):
    assert P.plan_info(m, n, dtype=P.F32)["work_items"] == _tri(n, 128)


@pytest.mark.parametrize("m,n", [(825, 2300), (1000, 3072), (2000, 3072), (600, 2048), (390, 2355), (256, 192)])
def test_f32_on_fine_tiles(m, n):
    assert P.plan_info(m, n, dtype=P.F32)["work_items"] > _tri(n, 128)


@pytest.mark.parametrize("m,n", [(7597, 3061), (7780, 2979), (7297, 3046), (8108, 2950), (7252, 3050)])
def test_f64_on_128_tiles(m, n):
    st = P.plan_info(m, n, dtype=P.F64)
    assert st["work_items"] % _tri(n, 128) == 0 and st["work_items"] // _tri(n, 128) == 7


@pytest.mark.parametrize("m,n", [(3001, 1203), (2121, 3652), (2368, 2777), (3979, 1492), (5984, 1887)])
def test_f64_on_fine_tiles(m, n):
    assert P.plan_info(m, n, dtype=P.F64)["work_items"] % _tri(n, 64) == 0
