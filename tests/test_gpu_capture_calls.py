"""Calls under stream capture: A A^t through its transpose takes one memory node
(replays against the eager result); least squares and the projection are
refused before anything is captured, and the capture goes on."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    return torch, P


def test_least_squares_and_projection_are_refused(env):
    torch, P = env
    print("case: refused under capture", flush=True)
    A = torch.rand((300, 40), dtype=torch.float64, device="cuda")
    B = torch.rand((300, 2), dtype=torch.float64, device="cuda")
    X = torch.empty((40, 2), dtype=torch.float64, device="cuda")
    Y = torch.empty((300, 2), dtype=torch.float64, device="cuda")
    P.normal_solve(A, B, X=X)
    P.project(A, B, out=Y)
    z = torch.zeros(10, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = []
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        for call in (lambda: P.normal_solve(A, B, X=X), lambda: P.project(A, B, out=Y)):
            try:
                call()
            except P.AtaError as e:
                got.append(e.status)
        z.add_(1.0)
    assert got == [3, 3]  # unsupported
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert bool((z == k + 1).all())


@pytest.mark.parametrize("m,n,f32", [(4300, 70, False), (4300, 300, True)])
def test_captured_row_products_through_the_transpose(env, m, n, f32):
    torch, P = env
    print("case: captured row products", m, n, f32, flush=True)
    dt = torch.float32 if f32 else torch.float64
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    A = torch.randint(-3, 4, (m, n), generator=gen, device="cuda").to(dt)
    ref = P.gram_rows(A)
    C = torch.zeros_like(ref)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        P.gram_rows(A, out=C)
    for _ in range(3):
        C.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        x = P.gram_rows(A)
        torch.cuda.synchronize()
        assert torch.equal(C, ref) and torch.equal(x, ref)
