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
