"""One-block solves with more right-hand sides than one launch holds (64 threads
each, less than 2^32 threads a launch).  Small integers, so every result is exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    yield torch, P
    torch.cuda.empty_cache()


def test_one_block_solve_with_2_26_right_hand_sides(env):
    torch, P = env
    n, r = 2, (1 << 26) + 3
    print("case: one-block solve", n, r, flush=True)
    L = torch.tensor([2.0, 1.0, 1.0], device="cuda")  # L = [2 0; 1 1], L L^t = [4 2; 2 2]
    x0 = (torch.arange(r, device="cuda") % 9 - 4).to(torch.float32)
    B = torch.stack([4.0 * x0 + 2.0, 2.0 * x0 + 2.0])  # X = (x0, 1)
    P.cholesky_solve(L, B, n)
    assert torch.equal(B[0], x0)
    assert bool((B[1] == 1.0).all())
