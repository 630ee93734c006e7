"""Budgets that hold a request's matrices and the partial tiles of its 128 x 128
plan but not those of its fastest plan: the request is still admitted (simulate
mode, no GPU)."""
import pytest

import paper_1902_02104_amd as P
from paper_1902_02104_amd.serving import Server


# parts: bytes of the partial tiles of the 128 x 128 plan
@pytest.mark.parametrize("m,n,dtype,parts", [(2876, 630, P.F64, 6350592), (114613, 18, P.F32, 165888),
                                             (168810, 16, P.F32, 131072)])
def test_requests_fit_as_on_128_tiles(m, n, dtype, parts):
    eb = 8 if dtype == P.F64 else 4
    budget = m * n * eb + P.tri(n) * eb + parts + (128 << 10)
    assert P.workspace_bytes(m, n, dtype=dtype) > parts + (128 << 10)
    with Server(budget, simulate_tflops=1.0) as s:
        t = s.submit(m, n, dtype)
        s.wait(t, timeout=30)
        s.release(t)
        assert s.stats()["rejected"] == 0
        with pytest.raises(P.AtaError):
            s.submit(2 * m, n, dtype)  # does not fit whatever the plan
