"""The bound of the kept scratch memory, reached with workspaces of known size
(A A^t of more than 4000 rows copies A^t), on one stream, on several, and by
streams that are idle."""
import ctypes
import time

import pytest

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture()
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02104_amd as P
    P.load()
    hip = ctypes.CDLL("libamdhip64.so.7")

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0] // MB

    P.release_caches()
    yield torch, P, hip, free
    P.release_caches()
    torch.cuda.empty_cache()


class _Stream:
    def __init__(self, torch, hip):
        self.hip, self.h = hip, ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(self.h), 1) == 0  # non-blocking
        self.s = torch.cuda.ExternalStream(self.h.value)

    def destroy(self):
        assert self.hip.hipStreamDestroy(self.h) == 0


def test_one_stream_makes_room(env):
    torch, P, hip, free = env
    print("case: scratch bound, one stream", flush=True)
    A = torch.zeros((4500, 15000), device="cuda")
    C = torch.empty(P.tri(4500), device="cuda")
    P.gram_rows(A[:, :64], out=C)
    P.release_caches()
    before = free()
    most = 0
    for k in (3000, 6000, 9000, 12000, 15000):  # copies of 51 to 257 MB, 772 in all
        P.gram_rows(A[:, :k], out=C)
        most = max(most, before - free())
        assert before - free() <= 512 + 64
    assert most >= 350
    P.release_caches()
    assert before - free() <= 64


def test_streams_share_the_bound(env):
    torch, P, hip, free = env
    print("case: scratch bound, several streams", flush=True)
    A = torch.zeros((4500, 9000), device="cuda")  # a copy of 154 MB a call
    outs = [torch.empty(P.tri(4500), device="cuda") for _ in range(8)]
    P.gram_rows(A[:, :64], out=outs[0])
    streams = [_Stream(torch, hip) for _ in range(8)]
    torch.cuda.synchronize()
    P.release_caches()
    before = free()
    for _ in range(2):
        for s, C in zip(streams, outs):
            P.gram_rows(A, out=C, stream=s.s)
    held = before - free()
    assert 350 <= held <= 512 + 64
    P.release_caches()
    assert before - free() <= 64
    for s in streams:
        s.destroy()


def test_blocks_of_idle_streams_go_back(env):
    torch, P, hip, free = env
    print("case: scratch of idle streams", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randint(-4, 5, (20000, 256), generator=gen, device="cuda").to(torch.float64)
    il = torch.tril_indices(256, 256, device="cuda")
    ref = (A.t().contiguous() @ A)[il[0], il[1]]
    out = torch.empty_like(ref)
    one = P.workspace_bytes(20000, 256) // MB
    assert one >= 2
    torch.cuda.synchronize()
    P.release_caches()
    before = free()
    idle = [_Stream(torch, hip) for _ in range(80)]
    s = _Stream(torch, hip)
    for x in idle:
        P.gram(A, out=out, stream=x.s)
        torch.cuda.synchronize()
    assert torch.equal(out, ref)
    held = before - free()
    assert held >= min(448, 60 * one)
    time.sleep(1.2)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        P.gram(A, out=out, stream=s.s)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    assert held - (before - free()) >= 100  # the quarter that a library stream waits for
    for x in idle + [s]:
        x.destroy()


def test_capture_survives_eager_calls_that_find_no_room(env):
    """A capture on one stream while an eager call on another takes the place of
    idle blocks, which must not wait for the device.  (HIP calls by hand: a
    capture that ends with an error is an error code here.)"""
    torch, P, hip, free = env
    print("case: scratch beside a capture", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    A = torch.randint(-4, 5, (20000, 256), generator=gen, device="cuda").to(torch.float64)
    il = torch.tril_indices(256, 256, device="cuda")
    ref = (A.t().contiguous() @ A)[il[0], il[1]]
    C, D = torch.empty_like(ref), torch.zeros_like(ref)
    idle = [_Stream(torch, hip) for _ in range(80)]
    other, s = _Stream(torch, hip), _Stream(torch, hip)
    P.gram(A, out=C)  # the plan is made
    for x in idle:
        P.gram(A, out=C, stream=x.s)
    torch.cuda.synchronize()
    time.sleep(1.2)
    before = free()
    for mode in (0, 1, 2):
        C.zero_()
        D.zero_()
        torch.cuda.synchronize()
        graph, exe = ctypes.c_void_p(), ctypes.c_void_p()
        assert hip.hipStreamBeginCapture(s.h, mode) == 0
        try:
            P.gram(A, out=C, stream=other.s)
            P.gram(A, out=D, stream=s.s)
        finally:
            ended = hip.hipStreamEndCapture(s.h, ctypes.byref(graph))
            hip.hipGetLastError()
        assert ended == 0
        assert hip.hipGraphInstantiate(ctypes.byref(exe), graph, None, None, ctypes.c_size_t(0)) == 0
        for _ in range(3):
            D.zero_()
            torch.cuda.synchronize()
            assert hip.hipGraphLaunch(exe, s.h) == 0
            torch.cuda.synchronize()
            assert torch.equal(D, ref) and torch.equal(C, ref)
        assert hip.hipGraphExecDestroy(exe) == 0 and hip.hipGraphDestroy(graph) == 0
    assert free() - before >= 90  # idle blocks went back
    for x in idle + [other, s]:
        x.destroy()
