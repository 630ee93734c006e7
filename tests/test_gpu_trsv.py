"""GPU parity of the triangular solves that run as one chained launch per
direction, at the edges of their 64-row blocks, 128-row workgroups and groups
of right-hand sides, against the CPU oracle.  Integer factors with diagonal
entries in {1, 2, 4} and integer solutions: every product, sum and reciprocal
is exact, so results must equal the oracle bit for bit in FP64 and FP32."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    return torch, P


def _case(orc, n, r, seed):
    L0 = synthetic.integer_factor(n, seed)
    X0 = synthetic.integer(n, r, seed + 1)
    return orc.pack(L0), (L0 @ (L0.T @ X0)), X0


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 191, 192, 193, 257, 449])
@pytest.mark.parametrize("f32", [False, True])
def test_chained_solve_exact(env, orc, n, f32):
    torch, P = env
    dt = torch.float32 if f32 else torch.float64
    for r in (1, 2, 3, 4, 5):
        print("case: chained solve", n, r, f32, flush=True)
        Lp, Bn, X0 = _case(orc, n, r, 1000 + n)
        L = torch.from_numpy(Lp).to(dt).cuda()
        B = torch.full((n, r + 2), 77.0, dtype=dt, device="cuda")
        B[:, :r] = torch.from_numpy(Bn).to(dt)
        P.cholesky_solve(L, B[:, :r], n)
        assert np.array_equal(B[:, :r].cpu().double().numpy(), X0)
        assert bool((B[:, r:] == 77.0).all())


def test_chained_solve_passes_streams_and_capture(env, orc):
    """More right-hand sides than one pass, two solves at once on two streams,
    and a captured solve replayed with other work between the replays."""
    torch, P = env
    print("case: chained solve passes, streams, capture", flush=True)
    n, r = 200, 131
    Lp, Bn, X0 = _case(orc, n, r, 77)
    L = torch.from_numpy(Lp).cuda()
    B0 = torch.from_numpy(Bn).cuda()
    X = torch.from_numpy(X0).cuda()
    Bs = [B0.clone(), B0.clone()]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(3):
        for s, B in zip(streams, Bs):
            with torch.cuda.stream(s):
                B.copy_(B0)
                P.cholesky_solve(L, B, n)
    torch.cuda.synchronize()
    assert torch.equal(Bs[0], X) and torch.equal(Bs[1], X)
    B = torch.empty_like(B0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.copy_(B0)
        P.cholesky_solve(L, B, n)
    for _ in range(4):
        B.zero_()
        torch.randn(1000, device="cuda").sum().item()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(B, X)
