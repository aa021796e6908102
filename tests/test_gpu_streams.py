"""The binding launches on the calling thread's current stream."""
import threading

import pytest

from paper_2402_04902_amd import binding

pytestmark = pytest.mark.gpu


def test_stream_handle_follows_torch():
    import torch
    default = torch.cuda.current_stream().cuda_stream
    assert binding._stream() == default
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert binding._stream() == s.cuda_stream == torch.cuda.current_stream().cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append((binding._stream(), torch.cuda.current_stream().cuda_stream)))
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1]  # (streams are per thread)
    assert binding._stream() == default


def test_calls_are_ordered_with_a_side_stream():
    """Inputs written on a side stream right before the call: right only if the call is queued on that stream too."""
    import torch
    from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec
    spec = LayerSpec("stream", 3, 1024, 264, 8, 16.0, 4, 128, DTYPE_BF16)
    desc = binding.make_desc(spec)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1)
    X = torch.randn((3, 1024), generator=gen, device="cuda:0").bfloat16()
    packed = torch.randint(-2**31, 2**31 - 1, (264, 128), generator=gen, dtype=torch.int32, device="cuda:0")
    scale, zero = torch.full((264, 8), 0.01, device="cuda:0"), torch.full((264, 8), 0.02, device="cuda:0")
    want, got, late = (torch.zeros((3, 264), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
    binding.l4q_quantized_forward(desc, X, packed, scale, zero, want)
    torch.cuda.synchronize()
    s, Xs = torch.cuda.Stream(), torch.zeros_like(X)
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        torch.cuda._sleep(2_000_000)
        Xs.copy_(X)
        binding.l4q_quantized_forward(desc, Xs, packed, scale, zero, got)
        late.copy_(got)
    s.synchronize()
    assert torch.equal(late, want) and bool(want.abs().sum() > 0)
