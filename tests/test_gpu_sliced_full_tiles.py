"""Forward and dX products in k-slices of 256 x 256 macro tiles (weights too large for the memory-side cache): ragged tokens
and rows, k ranges that end inside a stage, against binary64 products of the weight that the library's own codes give."""
import pytest

from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

pytestmark = pytest.mark.gpu


def test_sliced_full_tiles():
    import torch
    from paper_2402_04902_amd import binding
    T, o, i, r, g, bits = 408, 8272, 8216, 8, 8, 4
    spec = LayerSpec("sliced_full", T, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device=dev) * std).bfloat16()
    X, dY, W0, A, B = normal(T, i), normal(T, o, std=1e-2), normal(o, i, std=0.02), normal(r, i, std=0.01), normal(o, r, std=1e-3)
    G = i // g
    scale = torch.full((o, G), 0.006, device=dev)
    zero = torch.randn((o, G), generator=gen, device=dev) * 2e-3
    desc = binding.make_desc(spec)
    fwd, bwd = binding.l4q_workspace_bytes(desc)
    pad = [(n + 31) // 32 * 32 for n in (o, i)]
    # three slices of each output, as far as the workspace tells (the backward one's holds them last)
    assert fwd - o * pad[1] * 2 >= 3 * T * o * 4 and bwd >= i * pad[0] * 2 + 3 * T * i * 4
    ws = torch.empty(max(fwd, bwd), dtype=torch.uint8, device=dev)
    Y, dX = torch.empty_like(dY), torch.empty_like(X)
    grads = [torch.empty(s, device=dev) for s in ((r, i), (o, r), (o, G), (o, G))]
    binding.l4q_forward(desc, X, W0, A, B, scale, zero, Y, ws)
    binding.l4q_backward(desc, X, dY, W0, A, B, scale, zero, dX, *grads, ws)
    codes = torch.empty((o, i), dtype=torch.int8, device=dev)
    binding.l4q_export_codes(desc, W0, A, B, scale, zero, codes)
    torch.cuda.synchronize()
    # Wq: one rounding of code s + b to binary32 (fused), then to bfloat16
    Wq = codes.double() * scale.double().repeat_interleave(g, 1) + zero.double().repeat_interleave(g, 1)
    Wq = Wq.float().bfloat16().double()
    for name, got, want in (("Y", Y.double(), X.double() @ Wq.t().contiguous()), ("dX", dX.double(), dY.double() @ Wq)):
        # one rounding to bfloat16 (2^-8 of a value at most) on binary32 sums of 8272 terms, whose error stays below
        # sqrt(8272) 2^-24 = 5e-6 of the sum's rms; 1e-4 for the worst of 3.4e6 elements
        bound = want.abs() * 2.0 ** -8 + 1e-4 * want.square().mean().sqrt()
        worst = ((got - want).abs() / bound).max().item()
        assert worst <= 1.0, (name, worst)
