"""Quantized forward of up to 64 tokens in one pass, of more in several (l4q_infer_blocks.hip), at the edges of its tiles, macros, steps, slices and
waves (the form each case takes is checked on the host in test_blocks_route.py), against binary64; what is not finite stays
where it belongs: a token in its row, a scale in its row of weights."""
import pytest

from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec
from test_blocks_route import GPU_CASES, GPU_PASSES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,i,o,bits,g", [c[0] for c in GPU_CASES + GPU_PASSES])
def test_blocks(T, i, o, bits, g):
    quantized_forward_against_binary64(T, i, o, bits, g)


def quantized_forward_against_binary64(T, i, o, bits, g):
    import torch
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"blocks_{T}x{i}x{o}_{bits}b_g{g}", T, i, o, 8, 16.0, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(T + i + bits)
    codes = torch.randint(0, 1 << bits, (o, i), generator=gen, device=dev)
    place = torch.arange(bits, device=dev)
    bitsof = (codes.unsqueeze(2) >> place & 1).view(o, i * bits // 32, 32).long()
    words = (bitsof << torch.arange(32, device=dev)).sum(2)
    packed = torch.where(words >= 1 << 31, words - (1 << 32), words).int()
    scale = torch.rand(o, i // g, generator=gen, device=dev) * 0.01 + 0.002
    zero = torch.randn(o, i // g, generator=gen, device=dev) * 0.01
    X = torch.randn(T, i, generator=gen, device=dev).bfloat16()
    W = (codes - (1 << (bits - 1))).double() * scale.double().repeat_interleave(g, 1) + zero.double().repeat_interleave(g, 1)
    want = X.double() @ W.t().contiguous()
    bad_token, bad_row = T // 2 if T > 1 else T, o - 3   # (a single token has no NaN)
    X[bad_token:bad_token + 1, i - 1] = float("nan")
    scale[bad_row, 0] = float("inf")
    desc = binding.make_desc(spec)
    ws = torch.empty(max(256, binding.l4q_quantized_forward_workspace_bytes(desc)), dtype=torch.uint8, device=dev)
    for workspace in (ws, None):
        Y = torch.full((T, o), 7.0, dtype=torch.bfloat16, device=dev)
        binding.l4q_quantized_forward(desc, X, packed, scale, zero, Y, *([workspace] if workspace is not None else []))
        torch.cuda.synchronize()
        got = Y.double()
        assert torch.isnan(got[bad_token:bad_token + 1]).all()
        assert not torch.isfinite(got[:, bad_row]).any()
        rows, cols = torch.arange(T, device=dev) != bad_token, torch.arange(o, device=dev) != bad_row
        g2, w2 = got[rows][:, cols], want[rows][:, cols]
        # exact codes and binary32 sums.  The sums carry X (u + 128): at 4 bits 136 of every code's 4.6 rms, terms 30 times the
        # result's, each off by up to 2^-24 of the partial sum they join: 30 sqrt(i) 2^-24 < 4e-4 of a value at i <= 32768.  And one
        # rounding of Y to bfloat16, at most 2^-8 of a value, 2^-9 / sqrt(3) = 1.1e-3 rms at the top of its binade, twice that at the bottom.
        bound = w2.abs() * 2.0 ** -8 + 1e-3 * w2.square().mean().sqrt()
        assert ((g2 - w2).abs() / bound).max().item() <= 1.0
        assert ((g2 - w2).norm() / w2.norm()).item() <= 2.2e-3
