"""Solves in which a value overflows or is infinite: column by column, a solved
value reaches the rows after it in the order of the substitution and no row
that is solved already.  The reference runs the same column steps in numpy."""
import numpy as np
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


def _solve(L, b):
    x = b.copy()
    n = len(x)
    with np.errstate(all="ignore"):
        for c in range(n):
            x[c] = x[c] / L[c, c]
            x[c + 1:] -= L[c + 1:, c] * x[c]
        for c in range(n - 1, -1, -1):
            x[c] = x[c] / L[c, c]
            x[:c] -= L[c, :c] * x[c]
    return x


def _check(env, orc, L, b):
    torch, P = env
    t = torch.from_numpy(orc.pack(L)).to(torch.from_numpy(b).dtype).cuda()
    for r in (1, 2, 3):
        B = torch.from_numpy(np.repeat(b[:, None], r, 1).copy()).cuda()
        P.cholesky_solve(t, B, len(b))
        want = _solve(L.astype(b.dtype), b)
        got = B.cpu().numpy()
        for q in range(r):
            assert np.array_equal(got[:, q], want, equal_nan=True), (r, q, got[:8, q], want[:8])


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("n,p,q", [(7, 3, 5), (64, 20, 50), (70, 3, 5), (70, 66, 68), (200, 130, 140),
                                   (200, 70, 190), (300, 5, 299)])
def test_overflow_in_the_back_substitution(env, orc, n, p, q, f32):
    """x_p overflows in the back substitution: the rows after p keep their
    finite values.  Diagonal of ones; row q meets column p with a large entry,
    and a one below every diagonal entry up to p carries x_p to the rows
    before."""
    print("case: overflow", n, p, q, f32, flush=True)
    dt = np.float32 if f32 else np.float64
    big = 2.0 ** 70 if f32 else 2.0 ** 600
    L = np.eye(n)
    L[q, p] = big
    for i in range(1, p + 1):
        L[i, i - 1] = 1.0
    b = np.zeros(n)
    b[q] = big
    b[q + 1:] = 3.0
    b[p + 1:q] = 2.0
    want = _solve(L.astype(dt), b.astype(dt))
    assert np.isinf(want[p]) and np.isfinite(want[p + 1:]).all()
    _check(env, orc, L, b.astype(dt))


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("n,p", [(2, 0), (40, 7), (70, 69), (130, 64), (200, 199)])
def test_infinite_right_hand_side(env, orc, n, p, f32):
    """An infinite entry in a chain of neighbours: signs follow the steps."""
    print("case: infinite entry", n, p, f32, flush=True)
    L = np.eye(n) + np.diag(np.ones(n - 1), -1)
    b = np.zeros(n)
    b[p] = np.inf
    _check(env, orc, L, b.astype(np.float32 if f32 else np.float64))


@pytest.mark.parametrize("n", [64, 100, 200])
def test_reciprocal_out_of_range(env, orc, n):
    """A diagonal entry whose reciprocal overflows."""
    print("case: tiny diagonal", n, flush=True)
    L = np.eye(n)
    L[n - 2, n - 2] = 2.0 ** -1074
    L[n - 1, n - 2] = 1.0
    _check(env, orc, L, np.ones(n))
