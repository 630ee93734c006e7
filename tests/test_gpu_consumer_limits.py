"""Sizes of A^t B whose launches pass the grid limits of HIP (grid x block
threads of a dimension below 2^32).  Small integers, so
every result is exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    yield torch, P
    P.release_caches()
    torch.cuda.empty_cache()


def test_atb_with_2_28_results(env):
    torch, P = env
    m, n, r = 65, 16384, 16384
    print("case: atb", m, n, r, flush=True)
    A = (torch.arange(m * n, device="cuda") % 7 - 3).to(torch.float32).reshape(m, n)
    B = (torch.arange(m * r, device="cuda") % 5 - 2).to(torch.float32).reshape(m, r)
    out = P.atb(A, B)
    for j in (0, 1, 63, 64, 8191, 8192, 16382, 16383):
        assert torch.equal(out[j], (A[:, j].double()[:, None] * B.double()).sum(0).float()), j
    ca, cb = A.double().sum(1), B.double().sum(1)
    assert out.sum(dtype=torch.float64).item() == (ca * cb).sum().item()


def test_atb_with_2_30_columns(env):
    torch, P = env
    m, n = 1, (1 << 30) + 70
    print("case: atb", m, n, 1, flush=True)
    A = torch.empty((m, n), dtype=torch.float32, device="cuda")
    A[0, :] = 1.0
    A[0, -100:] = torch.arange(100, device="cuda")
    B = torch.full((m, 1), 3.0, dtype=torch.float32, device="cuda")
    out = P.atb(A, B)
    assert out.shape == (n, 1)
    assert torch.equal(out[-100:, 0], 3.0 * torch.arange(100, dtype=torch.float32, device="cuda"))
    assert bool((out[:-100] == 3.0).all())
