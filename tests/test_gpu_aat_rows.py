"""GPU parity of A A^t on fine tiles that read the rows of A as they are, at the
edges of their tiles (32 and 64 rows), stages and parts, over row strides whose
padding holds NaN.  Integer inputs of magnitude at most 4: every sum is an
exact integer below 2^24.  Uniform inputs: sums of n terms differ by at most
n u relative to sqrt(C_ii C_jj) in any order (u = 2^-53 for FP64; FP32
accumulates at most 512 terms in FP32, then in FP64, and rounds the result
once: 514 u more with u = 2^-24), on both sides of the comparison."""
import pytest

pytestmark = pytest.mark.gpu

# (rows, row length): one and several tiles and parts, remainders of the
# stages (8, 16 and 32 elements) and of the 16-byte chunks
SHAPES = [(1, 1), (31, 7), (32, 33), (33, 130), (64, 127), (65, 2049), (97, 3001), (200, 515), (300, 5003), (40, 20011),
          (700, 1100), (1000, 4099), (1481, 648)]


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("form", ["f64", "f32", "f32_out64"])
def test_aat_rows(m, n, form):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    dtype = {"f64": P.F64, "f32": P.F32, "f32_out64": P.F32 | P.OUT_F64}[form]
    dt = torch.float64 if form == "f64" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    il = torch.tril_indices(m, m, device="cuda")
    Ai = torch.randint(-4, 5, (m, n), generator=gen, device="cuda").to(dt)
    Au = torch.rand((m, n), generator=gen, device="cuda", dtype=torch.float64).mul_(2).sub_(1).to(dt)
    ref = (Ai.double() @ Ai.double().t().contiguous())[il[0], il[1]]
    full = Au.double() @ Au.double().t().contiguous()
    d = full.diagonal().sqrt()
    refu, scale = full[il[0], il[1]], d[il[0]] * d[il[1]]
    tol = 2 * n * 2.0 ** -53 + (0 if form == "f64" else 514 * 2.0 ** -24)
    for pad in (0, 1, 5):
        print("case: aat rows", m, n, form, pad, flush=True)
        buf = torch.full((m, n + pad), float("nan"), device="cuda", dtype=dt)
        A = buf[:, :n]
        A.copy_(Ai)
        assert torch.equal(P.gram_rows(A, dtype=dtype).double(), ref)
        A.copy_(Au)
        got = P.gram_rows(A, dtype=dtype)
        assert torch.equal(got, P.gram_rows(A, dtype=dtype))
        assert float(((got.double() - refu).abs() / scale).max()) <= tol
