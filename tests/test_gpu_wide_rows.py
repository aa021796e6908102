"""Forward and dX products with the caller's operand loaded 64 k-values at a time: rows that end at every kind of place inside
such a unit (and inside the 32 k-values that the weight comes in), one unit to more than the ring holds, in each tile form,
against binary64 products of the weight that the library's own codes give; a NaN token stays in its row."""
import pytest

from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n", [(130, 264), (300, 16400), (4096, 4096)])  # 128 x 128, 128 x 256, 256 x 256 tiles
@pytest.mark.parametrize("k", [8, 32, 40, 64, 72, 96, 104, 160, 320, 696])
@pytest.mark.parametrize("transposed", [False, True])  # Y (k = in-features), dX (k = out-features)
def test_wide_rows(T, n, k, transposed):
    import torch
    from paper_2402_04902_amd import binding
    o, i = (k, n) if transposed else (n, k)
    r, g, bits = 8, 8, 4
    spec = LayerSpec(f"wide_{T}x{i}x{o}", T, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(k)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device=dev) * std).bfloat16()
    X, dY, W0, A, B = normal(T, i), normal(T, o, std=1e-2), normal(o, i, std=0.02), normal(r, i, std=0.01), normal(o, r, std=1e-3)
    nan_row = T - 2
    (dY if transposed else X)[nan_row] = float("nan")
    G = i // g
    scale = torch.full((o, G), 0.006, device=dev)
    zero = torch.randn((o, G), generator=gen, device=dev) * 2e-3
    desc = binding.make_desc(spec)
    ws = torch.empty(max(binding.l4q_workspace_bytes(desc)), dtype=torch.uint8, device=dev)
    Y, dX = torch.empty_like(dY), torch.empty_like(X)
    if transposed:
        grads = [torch.empty(s, device=dev) for s in ((r, i), (o, r), (o, G), (o, G))]
        binding.l4q_backward(desc, X, dY, W0, A, B, scale, zero, dX, *grads, ws)
    else:
        binding.l4q_forward(desc, X, W0, A, B, scale, zero, Y, ws)
    codes = torch.empty((o, i), dtype=torch.int8, device=dev)
    binding.l4q_export_codes(desc, W0, A, B, scale, zero, codes)
    torch.cuda.synchronize()
    Wq = codes.double() * scale.double().repeat_interleave(g, 1) + zero.double().repeat_interleave(g, 1)
    Wq = Wq.float().bfloat16().double()
    got, want = (dX.double(), dY.double() @ Wq) if transposed else (Y.double(), X.double() @ Wq.t().contiguous())
    assert torch.isnan(got[nan_row]).all()
    keep = torch.arange(T, device=dev) != nan_row
    got, want = got[keep], want[keep]
    # one rounding to bfloat16 (2^-8 of a value at most) on binary32 sums of k <= 696 terms, each at most a unit (2^-24) of the
    # partial sum off: below sqrt(696) 2^-24 = 1.6e-6 of the sum's rms in the mean, 1e-4 for the worst element
    bound = want.abs() * 2.0 ** -8 + 1e-4 * want.square().mean().sqrt()
    assert ((got - want).abs() / bound).max().item() <= 1.0
