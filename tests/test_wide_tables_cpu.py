"""Workspace of the reduced-precision plans: a plan holds the wide tiles of its
own form alone."""
import pytest

import paper_1902_02104_amd as P


@pytest.mark.parametrize("m,n", [(104861, 416), (133243, 433), (152277, 416), (169506, 455)])
def test_e4m3_plans_hold_no_bfloat16_parts(m, n):
    """The e4m3 copy of A, its scales and up to two rounds of 512 FP64 partial
    tiles of K parts; no last round of 256 x 128 bfloat16 tiles, whose partial
    tiles are another 64 MB."""
    ldt = (m + 127) // 128 * 128
    parts = 1024 * 128 * 128 * 8
    assert P.workspace_bytes(m, n, dtype=P.F32_FP8) <= n * ldt + 4 * n * (m // 256 + 2) + parts + 4096
