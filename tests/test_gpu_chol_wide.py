"""GPU parity of the Cholesky factor where the trailing update runs on 128 x 128
tiles (from 4737 columns on), and of a captured factor on one stream and on two.
Integer factors with diagonal entries in {1, 2, 4}: every pivot, product and sum
is exact, so results must equal the known factor bit for bit."""
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


@pytest.mark.parametrize("n", [4737, 4801, 5000])
@pytest.mark.parametrize("f32", [False, True])
def test_factor_exact_on_128_tiles(env, orc, n, f32):
    torch, P = env
    print("case: factor on 128 x 128 tiles", n, f32, flush=True)
    dt = torch.float32 if f32 else torch.float64
    L0 = synthetic.integer_factor(n, 70 + n)
    Cf = L0 @ L0.T
    assert np.abs(Cf).max() < 2.0 ** 24
    C = torch.from_numpy(orc.pack(Cf)).to(dt).cuda()
    info = torch.full((1,), -3, dtype=torch.int32, device="cuda")
    P.cholesky(C, n, info=info)
    assert int(info.item()) == 0
    assert torch.equal(C, torch.from_numpy(orc.pack(L0)).to(dt).cuda())


@pytest.mark.parametrize("n", [64, 700, 2500])
@pytest.mark.parametrize("f32", [False, True])
def test_captured_factor(env, orc, n, f32):
    """Replays with an eager factor and a synchronisation between them; 2500
    columns take the helper stream into the capture."""
    torch, P = env
    print("case: captured factor", n, f32, flush=True)
    dt = torch.float32 if f32 else torch.float64
    L0 = synthetic.integer_factor(n, 90 + n)
    C0 = torch.from_numpy(orc.pack(L0 @ L0.T)).to(dt).cuda()
    L = torch.from_numpy(orc.pack(L0)).to(dt).cuda()
    X, Y = C0.clone(), C0.clone()
    info = torch.full((1,), -3, dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        P.cholesky(X, n, info=info)  # the helper stream exists before the capture
        s.synchronize()
        assert torch.equal(X, L)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            X.copy_(C0)
            P.cholesky(X, n, info=info)
        for _ in range(4):
            X.zero_()
            info.fill_(-3)
            g.replay()
            Y.copy_(C0)
            P.cholesky(Y, n)
            torch.cuda.synchronize()
            assert torch.equal(X, L) and torch.equal(Y, L) and int(info.item()) == 0
