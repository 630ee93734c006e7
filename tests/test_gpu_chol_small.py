"""GPU parity of the Cholesky factor of a single block at the edges of its groups
of 16 columns.  Integer factors with diagonal entries in {1, 2, 4}: results must
equal the known factor bit for bit, up to the first bad pivot."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("f32", [False, True])
def test_single_block(orc, n, f32):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    print("case: single block", n, f32, flush=True)
    dt = torch.float32 if f32 else torch.float64
    L0 = synthetic.integer_factor(n, 300 + n)
    for p in [-1] + sorted({0, n // 2, n - 1}):
        Cf = L0 @ L0.T
        if p >= 0:
            Cf[p, p] -= L0[p, p] ** 2
        buf = torch.full((P.tri(n) + 64,), 7.0, dtype=dt, device="cuda")
        buf[: P.tri(n)] = torch.from_numpy(orc.pack(Cf)).to(dt).cuda()
        info = torch.full((1,), -3, dtype=torch.int32, device="cuda")
        P.cholesky(buf[: P.tri(n)], n, info=info)
        got = buf.cpu().double().numpy()
        assert int(info.item()) == p + 1
        k = P.tri(n if p < 0 else p)
        assert np.array_equal(got[:k], orc.pack(L0)[:k])
        assert (got[P.tri(n):] == 7.0).all()
