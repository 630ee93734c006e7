"""Bfloat16-pair products whose tables and copies fill the fixed scratch array
of the calls that allocate nothing."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(3072, 5435), (4480, 3728), (4608, 3625), (7040, 2373)])
def test_products_that_fill_the_array(m, n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    print("case: full scratch array", m, n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(m)
    A = torch.randint(-3, 4, (m, n), generator=gen, device="cuda").to(torch.float32)
    C, used = P.gram_noalloc(A, torch.empty(P.tri(n), device="cuda"), dtype=P.F32_BF16X3)
    assert (64 << 20) - 16384 < used <= 64 << 20
    assert torch.equal(C, P.gram(A))
