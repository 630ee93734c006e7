"""Outputs that share memory with an input: every input is read before the
output is written.  Small integers, so every result is exact."""
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


def _ints(torch, m, n, dt, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-3, 4, (m, n), generator=gen, device="cuda").to(dt)


@pytest.mark.parametrize("n", [65, 4000, 128000])
@pytest.mark.parametrize("dt", ["float32", "float64"])
def test_atb_over_its_right_hand_side(env, n, dt):
    """B in the first rows of the output: one chunk of rows, many workgroups."""
    torch, P = env
    dt = getattr(torch, dt)
    m = 64
    for r in (1, 5, 16, 33):
        print("case: atb in place", m, n, r, dt, flush=True)
        A = _ints(torch, m, n, dt, n + r)
        X = torch.zeros((n, r), dtype=dt, device="cuda")
        X[:m] = _ints(torch, m, r, dt, r)
        want = P.atb(A, X[:m].clone())
        P.atb(A, X[:m], out=X)
        assert torch.equal(X, want)


@pytest.mark.parametrize("m,n", [(40, 30), (1000, 512), (1500, 1000), (300, 20000)])
@pytest.mark.parametrize("dt", ["float32", "float64"])
def test_row_products_over_their_input(env, m, n, dt):
    """lower(A A^t) into A's own memory."""
    torch, P = env
    dt = getattr(torch, dt)
    print("case: row products in place", m, n, dt, flush=True)
    A = _ints(torch, m, n, dt, m + n)
    buf = torch.zeros(max(m * n, P.tri(m)), dtype=dt, device="cuda")
    buf[: m * n] = A.reshape(-1)
    want = P.gram_rows(A)
    P.gram_rows(buf[: m * n].reshape(m, n), out=buf[: P.tri(m)])
    assert torch.equal(buf[: P.tri(m)], want)


def test_wide_atb_over_its_right_hand_side(env):
    """2^28 results of one chunk through the separate sum, which has sixteen
    threads for each: more than a grid dimension holds."""
    torch, P = env
    m, n, r = 64, 16384, 16384
    print("case: wide atb in place", m, n, r, flush=True)
    A = _ints(torch, m, n, torch.float32, 1)
    X = torch.zeros((n, r), dtype=torch.float32, device="cuda")
    X[:m] = _ints(torch, m, r, torch.float32, 2)
    want = P.atb(A, X[:m].clone())
    P.atb(A, X[:m], out=X)
    assert torch.equal(X, want)
    del X, want
    P.release_caches()
    torch.cuda.empty_cache()
