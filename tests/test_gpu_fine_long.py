"""Fine tiles at the most rows the entry points take: a column of 2^31 - 1 ones
(8.6 GB in FP32).  Its square sum is 2^31 - 1; blocks of 512 rows are exact in
FP32 and their sums in FP64."""
import pytest

pytestmark = pytest.mark.gpu


def test_every_row_of_the_longest_column_counts():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    m = 2**31 - 1
    print("case: fine tiles", m, 1, flush=True)
    A = torch.ones((m, 1), dtype=torch.float32, device="cuda")
    C = P.gram(A, dtype=P.F32 | P.OUT_F64)
    assert C.dtype == torch.float64
    assert C.item() == float(m)
    del A
    torch.cuda.empty_cache()
