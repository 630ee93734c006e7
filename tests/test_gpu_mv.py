"""GPU parity of A^t B and A X over the widths, row tiles and column remainders
of their kernels.  Integer inputs of magnitude at most 4: every sum is an exact
integer below 2^24, so the results are exact in any order."""
import pytest

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 3, 4, 5, 8, 9, 16, 17, 33]


def _env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    return torch, P


@pytest.mark.parametrize("m,n", [(1, 1), (63, 65), (64, 64), (65, 130), (129, 1), (4100, 63), (9001, 200)])
@pytest.mark.parametrize("dt", ["float32", "float64"])
def test_atb_widths(m, n, dt):
    torch, P = _env()
    dt = getattr(torch, dt)
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    # strided operands whose padding holds NaN
    Ab = torch.full((m, n + 3), float("nan"), device="cuda", dtype=dt)
    Ab[:, :n] = torch.randint(-4, 5, (m, n), generator=gen, device="cuda").to(dt)
    for r in WIDTHS:
        print("case: atb", m, n, r, dt, flush=True)
        Bb = torch.full((m, r + 1), float("nan"), device="cuda", dtype=dt)
        Bb[:, :r] = torch.randint(-4, 5, (m, r), generator=gen, device="cuda").to(dt)
        ref = Ab[:, :n].double().t().contiguous() @ Bb[:, :r].double().contiguous()
        got = P.atb(Ab[:, :n], Bb[:, :r])
        torch.cuda.synchronize()
        assert torch.equal(got.double(), ref), r


@pytest.mark.parametrize("n", [1, 63, 64, 130, 333])
@pytest.mark.parametrize("dt", ["float32", "float64"])
def test_project_widths_exact(n, dt):
    """Columns of four stacked identities and seven zero rows: A^t A = 4 I, the
    factor is 2 I and the projection averages four rows of B, in quarters."""
    torch, P = _env()
    dt = getattr(torch, dt)
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = torch.cat([torch.eye(n, device="cuda", dtype=dt)] * 4 + [torch.zeros((7, n), device="cuda", dtype=dt)])
    for r in WIDTHS:
        print("case: project", n, r, dt, flush=True)
        B = torch.randint(-4, 5, (4 * n + 7, r), generator=gen, device="cuda").to(dt)
        ref = torch.zeros_like(B)
        ref[: 4 * n] = (B[: 4 * n].reshape(4, n, r).sum(0) / 4).repeat(4, 1)
        got = P.project(A, B)
        torch.cuda.synchronize()
        assert torch.equal(got, ref), r
