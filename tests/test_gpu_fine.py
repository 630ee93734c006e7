"""GPU parity of the fine-tile product (64 x 64 and 32 x 32 tiles with K split
over the waves of a workgroup and over workgroups) against the oracle, at the
edges of its tiles, stages and parts.  Integer inputs: every partial sum is an
integer below 2^24, so every form is exact.  Uniform inputs: sums of m terms
differ by at most m u relative to sqrt(C_ii C_jj) in any order (u = 2^-53 for
FP64; FP32 accumulates at most 512 rows in FP32, then in FP64, and rounds the
result once: 513 u + u with u = 2^-24)."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

# (m, n): remainders of the stages (8, 16, 32 rows) and tiles, one and several
# parts, part counts that are and are not multiples of eight, one column
SHAPES = [(1, 1), (7, 31), (33, 32), (65, 33), (127, 64), (130, 65), (257, 129), (512, 200), (1000, 100),
          (3001, 97), (5003, 300), (20011, 40), (40000, 1), (9000, 161), (700, 1100), (1500, 1203)]


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    return torch, P


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("form", ["f64", "f32", "f32_out64"])
def test_fine_tiles(env, orc, m, n, form):
    torch, P = env
    print("case: fine tiles", m, n, form, flush=True)
    dt = {"f64": P.F64, "f32": P.F32, "f32_out64": P.F32 | P.OUT_F64}[form]
    npdt = np.float64 if form == "f64" else np.float32
    Ai = synthetic.integer(m, n, 900 + m, dtype=npdt)
    ref = orc.classical(Ai.astype(np.float64))
    for lda in (n, n + 1, n + 5):  # odd and even strides; the pad holds NaN
        buf = torch.from_numpy(synthetic.with_lda(Ai, lda)).cuda()
        A = buf[:, :n]
        C = P.gram(A, dtype=dt)
        assert np.array_equal(C.cpu().double().numpy(), ref), lda
        # no K split over workgroups without an allocation
        out, _ = P.gram_noalloc(A, torch.empty_like(C), dtype=dt)
        assert np.array_equal(out.cpu().double().numpy(), ref), lda
    Au = synthetic.uniform(m, n, 901 + m, dtype=npdt)
    got = P.gram(torch.from_numpy(Au).cuda(), dtype=dt)
    again = P.gram(torch.from_numpy(Au).cuda(), dtype=dt)
    assert torch.equal(got, again)
    tol = m * 2.0 ** -53 if form == "f64" else m * 2.0 ** -53 + 514 * 2.0 ** -24
    assert orc.scaled_err(got.cpu().double().numpy(), orc.classical(Au.astype(np.float64)), n) <= tol


def test_fine_plans(env):
    """Where the rule takes fine tiles: few 128 x 128 tiles; partial tiles in
    the workspace when the rows are split; a larger product keeps the
    128 x 128 tiles."""
    torch, P = env
    assert P.plan_info(256, 192)["work_items"] == 21 and P.workspace_bytes(256, 192) == 0
    st = P.plan_info(262144, 64)
    assert st["combine_tasks"] == 1 and P.workspace_bytes(262144, 64) > 0
    assert P.plan_info(5000, 5000)["work_items"] == 820
