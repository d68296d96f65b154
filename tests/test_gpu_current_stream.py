"""The stream a call without one runs on: the calling thread's current stream
of its current device, on the default stream, inside a stream context and in
another thread, and a step issued there is ordered after that stream's work."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_follows_the_current_stream():
    import torch
    import paper_2606_23348_amd as gen

    def now():
        return gen._stream(None) or 0, torch.cuda.current_stream().cuda_stream or 0

    a, b = now()
    assert a == b
    s, seen = torch.cuda.Stream(), []
    with torch.cuda.stream(s):
        a, b = now()
        assert a == b == s.cuda_stream
        t = threading.Thread(target=lambda: seen.append(now()))
        t.start()
        t.join()
    assert seen[0][0] == seen[0][1]
    a, b = now()
    assert a == b and a != s.cuda_stream
    assert gen._stream(s) == s.cuda_stream and gen._stream(s.cuda_stream) == s.cuda_stream


def test_step_waits_for_its_stream():
    import torch
    import paper_2606_23348_amd as gen
    b, ref = (gen.Batch(64, 10, 10, 0, gen.make_params(0, 2), seed=3) for _ in range(2))
    b.sample(5, 0)
    ref.sample(5, 0)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    held = b.actions.clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        b.actions.zero_()
        x = torch.ones(4096, 4096, device="cuda")
        for _ in range(8):
            x = x @ x * 1e-4
        b.actions.copy_(held)          # after the products on this stream
        b.step()
    s.synchronize()
    ref.step()
    torch.cuda.synchronize()
    assert np.array_equal(b.buf.cpu().numpy(), ref.buf.cpu().numpy())
    assert np.array_equal(b.obs.cpu().numpy(), ref.obs.cpu().numpy())
