"""The scratch memory kept between calls: streams, threads, streams that are
destroyed and created again, capture, its bound and its release.  Integer
inputs, so every result is exact."""
import ctypes
import threading

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


def _case(torch, m, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randint(-4, 5, (m, n), generator=gen, device="cuda").to(torch.float32)
    il = torch.tril_indices(n, n, device="cuda")
    ref = (A.double().t().contiguous() @ A.double())[il[0], il[1]].float()
    torch.cuda.synchronize()
    return A, ref


def test_threads_and_streams(env):
    """Threads with a stream of their own, two streams each, shapes whose
    workspaces differ, while another thread releases the caches."""
    torch, P = env
    print("case: scratch threads", flush=True)
    cases = [_case(torch, 3000 + 500 * k, 70 + 30 * k, k) for k in range(4)]
    bad, stop = [], threading.Event()

    def work(k):
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        for it in range(40):
            A, ref = cases[(k + it) % 4]
            with torch.cuda.stream(streams[it % 2]):
                C = P.gram(A)
                ok = torch.equal(C, ref)
            if not ok:
                bad.append((k, it))

    def release():
        while not stop.wait(0.02):
            P.release_caches()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    r = threading.Thread(target=release)
    for t in ts + [r]:
        t.start()
    for t in ts:
        t.join()
    stop.set()
    r.join()
    assert not bad


def test_streams_created_again(env):
    """Streams that live for one call: a handle that comes back is another
    stream, ordered after the work of the old one on the kept block."""
    torch, P = env
    print("case: scratch recycled streams", flush=True)
    hip = ctypes.CDLL("libamdhip64.so.7")
    cases = [_case(torch, 4000 + 500 * k, 90 + 40 * k, 10 + k) for k in range(3)]
    outs = [(torch.empty_like(cases[it % 3][1]), cases[it % 3][1]) for it in range(30)]
    torch.cuda.synchronize()
    for it in range(30):
        h = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
        P.gram(cases[it % 3][0], out=outs[it][0], stream=torch.cuda.ExternalStream(h.value))
        assert hip.hipStreamDestroy(h) == 0
    torch.cuda.synchronize()
    for C, ref in outs:
        assert torch.equal(C, ref)


def test_capture_beside_kept_blocks(env):
    """A captured call does not use the kept blocks: eager calls between the
    replays write over them."""
    torch, P = env
    print("case: scratch capture", flush=True)
    A, ref = _case(torch, 5000, 120, 20)
    B, refb = _case(torch, 6000, 130, 21)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        C = P.gram(A)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            P.gram(A, out=C)
        for _ in range(4):
            C.zero_()
            g.replay()
            assert torch.equal(P.gram(B), refb)
            assert torch.equal(C, ref)


def test_bound_and_release(env):
    """Kept memory stays within half a gigabyte and goes back."""
    torch, P = env
    print("case: scratch bound", flush=True)
    P.release_caches()
    torch.cuda.synchronize()
    A = torch.zeros((1000, 40000), device="cuda")
    outs = [torch.empty(P.tri(1000), device="cuda")]
    P.gram_rows(A[:, :64], out=outs[0])
    torch.cuda.synchronize()
    P.release_caches()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for k in range(8):  # transposes of 20 to 160 MB, on one stream
        P.gram_rows(A[:, : 5000 * (k + 1)], out=outs[0])
    for k in range(8):  # and 80 MB on others
        P.gram_rows(A[:, :20000], out=outs[0], stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    slack = 64 << 20
    assert before - torch.cuda.mem_get_info()[0] <= (512 << 20) + slack
    P.release_caches()
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= slack
