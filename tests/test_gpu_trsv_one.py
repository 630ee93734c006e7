"""GPU parity of the single-block solves (n <= 64, one launch) at the edges of
their rows and right-hand sides.  Unit-diagonal integer factors and integer
solutions of magnitude at most 2: every intermediate value is an integer that
FP32 and FP64 hold, so the solves are exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 24, 33, 63, 64, 65])
@pytest.mark.parametrize("dt", ["float32", "float64"])
def test_one_block_solves_exact(n, dt):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    dt = getattr(torch, dt)
    gen = torch.Generator(device="cuda").manual_seed(n)
    # entries of the factor on two subdiagonals keep its products small
    L = torch.eye(n, device="cuda", dtype=torch.float64)
    for d in (1, 2):
        if n > d:
            L += torch.diag(torch.randint(-1, 2, (n - d,), generator=gen, device="cuda").double(), -d)
    il = torch.tril_indices(n, n, device="cuda")
    packed = L[il[0], il[1]].to(dt)
    for r in (1, 2, 7, 8, 9, 33, 130):
        print("case: one block", n, r, dt, flush=True)
        X = torch.randint(-2, 3, (n, r), generator=gen, device="cuda").double()
        buf = torch.full((n, r + 2), float("nan"), device="cuda", dtype=dt)
        buf[:, :r] = (L @ (L.t().contiguous() @ X)).to(dt)
        got = P.cholesky_solve(packed, buf[:, :r])
        torch.cuda.synchronize()
        assert torch.equal(got.double(), X), r
        assert bool(torch.isnan(buf[:, r:]).all())
