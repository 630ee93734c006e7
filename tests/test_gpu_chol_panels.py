"""GPU parity of the panel-blocked Cholesky factor at the edges of its steps
(64 columns), panels (256 columns), 64 x 64 and 128 x 128 update tiles and of
the single-launch update, against the CPU oracle.  Integer factors with
diagonal entries in {1, 2, 4}: every pivot is a power of four times one, every
product and sum an integer, so the factor must equal the oracle's bit for bit
in FP64 and FP32.  Pivots outside the fast root's range and non-positive ones
take the plain operations."""
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


def _factor(env, Cp, n, dt):
    torch, P = env
    C = torch.from_numpy(Cp).to(dt).cuda()
    info = torch.full((1,), -3, dtype=torch.int32, device="cuda")
    P.cholesky(C, n, info=info)
    return C.cpu().double().numpy(), int(info.item())


@pytest.mark.parametrize("n", [15, 16, 17, 64, 65, 255, 256, 257, 320, 383, 500, 513, 769, 2100, 2753])
@pytest.mark.parametrize("f32", [False, True])
def test_factor_exact_at_block_edges(env, orc, n, f32):
    torch, P = env
    print("case: factor exact", n, f32, flush=True)
    L0 = synthetic.integer_factor(n, 40 + n)
    # FP32: sums of 4 n stay exact; all partial sums are below 2^24
    C = orc.pack(L0 @ L0.T)
    got, info = _factor(env, C, n, torch.float32 if f32 else torch.float64)
    assert info == 0
    assert np.array_equal(got, orc.pack(L0))


@pytest.mark.parametrize("scale", [2.0 ** -480, 2.0 ** 480])
def test_factor_extreme_scales(env, orc, scale):
    """Pivots near the ends of the exponent range: scaling C by scale^2 scales
    L by scale, exactly for powers of two."""
    torch, P = env
    n = 150
    print("case: factor scale", scale, flush=True)
    L0 = synthetic.integer_factor(n, 9)
    got, info = _factor(env, orc.pack(L0 @ L0.T) * scale * scale, n, torch.float64)
    assert info == 0
    assert np.array_equal(got, orc.pack(L0) * scale)


@pytest.mark.parametrize("f32", [False, True])
def test_factor_bad_pivots_in_later_panels(env, orc, f32):
    torch, P = env
    n = 600
    L0 = synthetic.integer_factor(n, 11)
    for p in (255, 256, 300, 511, 512, 599):
        print("case: factor bad pivot", p, f32, flush=True)
        Cf = L0 @ L0.T
        Cf[p, p] -= L0[p, p] ** 2 + 1.0
        got, info = _factor(env, orc.pack(Cf), n, torch.float32 if f32 else torch.float64)
        assert info == p + 1
        assert np.array_equal(got[:orc.tri(p)], orc.pack(L0)[:orc.tri(p)])
