"""The stream a call without one runs on is torch's current stream of the current device, in every thread."""
import threading

import pytest


@pytest.mark.gpu
def test_default_stream_is_the_current_one():
    import torch
    from paper_1910_00178_amd import binding

    def current():
        return torch.cuda.current_stream().cuda_stream or None

    assert binding._stream(None) == current()           # binds the fast form
    side = torch.cuda.Stream()
    seen = {}
    with torch.cuda.stream(side):
        assert binding._stream(None) == current() == side.cuda_stream
        t = threading.Thread(target=lambda: seen.update(other=(binding._stream(None), current())))
        t.start()
        t.join()
        graph_stream = torch.cuda.Stream()
        with torch.cuda.stream(graph_stream):
            assert binding._stream(None) == graph_stream.cuda_stream
        assert binding._stream(None) == side.cuda_stream
    assert seen["other"][0] == seen["other"][1] != side.cuda_stream
    assert binding._stream(None) == current()
    assert binding._stream(side) == side.cuda_stream and binding._stream(0) is None


# The native calls look the stream up themselves: on the current stream of the calling thread, also after tests with stand-ins for it, and
# without the Python function having been asked.
@pytest.mark.gpu
def test_native_calls_find_the_current_stream():
    import ctypes

    import torch
    import paper_1910_00178_amd as ng
    from paper_1910_00178_amd import binding
    from test_calls import forget_streams
    M, N, K = 5, 70, 130
    A = torch.randint(0, 256, (M, K), dtype=torch.uint8, device="cuda")
    B = torch.randint(-128, 128, (N, K), dtype=torch.int8, device="cuda")
    want = (A.double() @ B.double().t()).int()
    ctx = ng.ngemm_create(0)
    packed = torch.empty(ng.ngemm_packed_b_bytes(K, N), dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b(ctx, K, N, B, K, packed, packed.numel())
    given = []

    def slow(*a):
        given.append(a)
        return ng.ngemm_run_u8s8s32.__wrapped__(*a)
    call = binding._calls.Call(slow, "run", ctypes.cast(binding._lib.ngemm_run_u8s8s32, ctypes.c_void_p).value)

    def run():
        C = torch.full((M, N), -1, dtype=torch.int32, device="cuda")
        call(ctx, M, A, K, 0, h, 0, C, N)
        torch.cuda.synchronize()
        assert torch.equal(C, want)

    def captured():                                      # a launch on any other stream is not in the graph
        C = torch.full((M, N), -1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            call(ctx, M, A, K, 0, h, 0, C, N)
        torch.cuda.synchronize()
        before = C.clone()
        g.replay()
        torch.cuda.synchronize()
        assert bool((before == -1).all()) and torch.equal(C, want)

    forget_streams()
    run()
    assert len(given) == 1                               # asked once, and bound by that
    run()
    with torch.cuda.stream(torch.cuda.Stream()):
        run()
    captured()
    failed = []

    def other_thread():
        try:
            run()
            captured()
        except BaseException as e:
            failed.append(e)
    t = threading.Thread(target=other_thread)
    t.start()
    t.join()
    assert not failed and len(given) == 1
    ng.ngemm_packed_b_free(h)
    ng.ngemm_destroy(ctx)
