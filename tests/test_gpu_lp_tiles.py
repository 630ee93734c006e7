"""GPU parity of the direct-to-LDS reduced-precision tiles: wide workgroup tiles
(256 x 128 bfloat16 pairs, 256 x 256 e4m3) and 128 x 128 ones, at the edges of
their tiles, stages, row blocks and K parts, in both output types.  Integer
inputs of magnitude at most 4: both formats hold them (a column's power-of-two
scale keeps four significand bits), every product is an integer and every
partial sum stays below 2^24, so the results are exact in any order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (m, n): below and at the smallest wide launches (bfloat16: 16 row panels of
# 256, e4m3: 23), last panels of 1 and 255 rows, stage remainders, K parts of
# the last round, short and long K, too few columns for wide tiles
SHAPES = [(1, 130), (40, 257), (136, 700), (8, 3841), (200, 4095), (1104, 4097), (72, 5633), (1160, 5887),
          (264, 6145), (66000, 300), (20008, 1025)]


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("form", ["bf16x3", "fp8"])
def test_lp_tiles_integer_exact(m, n, form):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    print("case: lp tiles", m, n, form, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1000 + m + n)
    A = torch.randint(-4, 5, (m, n), generator=gen, device="cuda").to(torch.float32)
    ref = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    for r in range(0, m, 8192):
        blk = A[r:r + 8192].double()
        ref += blk.t().contiguous() @ blk
    il = torch.tril_indices(n, n, device="cuda")
    ref = ref[il[0], il[1]]
    dt = P.F32_BF16X3 if form == "bf16x3" else P.F32_FP8
    for out in (0, P.OUT_F64):
        C = P.gram(A, dtype=dt | out, max_depth=0)
        torch.cuda.synchronize()
        assert torch.equal(C.double(), ref), (m, n, form, out)
        if m * n > 6000000:  # the copies do not fit the fixed scratch array
            continue
        C, _ = P.gram_noalloc(A, torch.full_like(C, float("nan")), dtype=dt | out, max_depth=0)
        torch.cuda.synchronize()
        assert torch.equal(C.double(), ref), (m, n, form, out, "noalloc")
