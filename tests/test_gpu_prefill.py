"""Quantized forward at prompt sizes (two-dimensional tiles): every tile shape and code width, token and row counts that end
inside a tile, one to eighteen sections of k (an odd count leaves half a zero-term pair), groups of half a section, one, two
and four in the shapes that have them, against the oracle; a NaN token stays in its row."""
import numpy as np
import pytest

from paper_2402_04902_amd import inputs
from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

from parity_util import compare_tensor, host_qparams, rel_fro
from plan_util import PASSES, TILES_128x128, TILES_128x256, TILES_64x128
from test_gpu_quantized_path import packed_on_gpu

pytestmark = pytest.mark.gpu


# (T, in, out, group), the tile shape that 2, 3, 4 and 8 bits take (tests/test_prompt_route.py keeps the two together)
CASES = [
    ((65, 128, 8, 128), (TILES_64x128,) * 4),     # one section, the second tile one token, eight rows
    ((129, 640, 264, 128), (TILES_64x128,) * 4),  # five sections
    ((100, 1152, 392, 64), (TILES_64x128, PASSES, TILES_64x128, TILES_64x128)),       # half sections
    ((130, 1536, 136, 512), (TILES_64x128,) * 4),    # groups of four sections
    ((401, 384, 5000, 128), (TILES_128x128,) * 4),   # three sections, ragged rows
    ((385, 512, 5128, 256), (TILES_128x128,) * 4),   # groups of two sections
    ((385, 1536, 5128, 512), (TILES_128x128,) * 4),  # ... of four
    ((385, 256, 5128, 64), (TILES_128x128, PASSES, TILES_128x128, TILES_128x128)),    # half sections, four of them
    ((257, 1152, 7944, 64), (TILES_128x128, PASSES, TILES_128x128, TILES_128x128)),   # ... eighteen
    ((385, 192, 5128, 64), (PASSES,) * 4),           # rows that are no multiple of 128
    ((641, 256, 8200, 128), (TILES_128x256, TILES_128x256, TILES_128x256, TILES_64x128)),  # one token in the last tile
    ((513, 640, 7496, 128), (TILES_128x256, TILES_128x256, TILES_128x256, TILES_64x128)),  # wide tiles of 192 rows, the last of 8 rows
    ((641, 384, 5896, 128), (TILES_128x256, TILES_128x256, TILES_128x256, TILES_64x128)),  # ... an odd count of sections, 136 rows in the last
]


@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("T,i,o,g", [c[0] for c in CASES])
def test_prefill(T, i, o, g, bits):
    import torch
    from oracle import l4q_oracle as O
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"prefill_{T}x{i}x{o}_{bits}b_g{g}", T, i, o, 8, 16.0, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=T + bits)
    s, b = host_qparams(spec, arrs, "asymm", 0.9)
    layer = binding.upload(spec, arrs, s, b)
    packed = packed_on_gpu(spec, layer)
    nan_row = T - 2
    layer.X[nan_row, i // 2] = float("nan")
    Y = torch.full_like(layer.Y, 7.0)
    binding.l4q_quantized_forward(layer.desc, layer.X, packed, layer.scale, layer.zero, Y)
    torch.cuda.synchronize()
    dec, _, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    ref = O.quantized_forward(arrs["X"], O.pack_codes(dec.codes, bits), s, b, bits, g)
    got = Y.double().cpu().numpy()
    assert np.isnan(got[nan_row]).all()
    keep = np.arange(T) != nan_row
    compare_tensor(spec.name, got[keep], ref[keep], 2e-2, 2e-2)
    # exact codes and binary32 sums: what is left is the rounding of Y to bfloat16, 2^-9 / sqrt(3) = 1.1e-3 rms of a value at
    # the top of its binade and up to twice that at the bottom (mean 1.7e-3)
    assert rel_fro(got[keep], ref[keep]) <= 2.2e-3


@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("T,o", [(129, 264), (401, 5000), (641, 8200)])  # 64 x 128, 128 x 128, 128 x 256 tiles
@pytest.mark.parametrize("i,col", [(640, 133), (896, 389)])  # five and seven sections of 128
def test_infinite_token_with_an_odd_section_count(i, col, T, o, bits):
    """Every weight positive: a token with +Inf has +Inf in all its outputs, wherever its section's sums lie when the last
    section's zero term, which has no partner, is added; no other token notices."""
    import torch
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"prefill_inf_{T}x{i}x{o}_{bits}b", T, i, o, 8, 16.0, bits, 128, DTYPE_BF16)
    print("case", spec.name, flush=True)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(bits)
    X = torch.rand((T, i), generator=gen, device="cuda:0").bfloat16()
    X[70, col] = float("inf")
    packed = torch.randint(-2**31, 2**31 - 1, (o, i * bits // 32), generator=gen, dtype=torch.int32, device="cuda:0")
    if bits == 8:
        packed |= -0x7E7E7E7F  # (codes above zero: eight bits enter the product without an offset)
    scale, zero = torch.full((o, i // 128), 0.01, device="cuda:0"), torch.full((o, i // 128), 10.0, device="cuda:0")
    Y = torch.zeros((T, o), dtype=torch.bfloat16, device="cuda:0")
    binding.l4q_quantized_forward(binding.make_desc(spec), X, packed, scale, zero, Y)
    torch.cuda.synchronize()
    assert (Y[70] == float("inf")).all()
    assert torch.isfinite(Y[torch.arange(T, device=Y.device) != 70]).all()
