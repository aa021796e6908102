"""The streaming pass's set-up forms (ranks that are multiples of 8, groups of 32 and more): packed codes of every width,
extremes across the wavefronts of a group, error sums with many and few partial pairs, at widths that end inside a strip
of 256 columns and heights that end inside a row block of 32, against the oracle (words and scales bit for bit)."""
import numpy as np
import pytest

from paper_2402_04902_amd import inputs
from paper_2402_04902_amd.inputs import DTYPE_BF16, DTYPE_F32, LayerSpec

from parity_util import host_qparams
from test_gpu_quantized_path import packed_on_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("i,o,r,g", [(32, 8, 8, 32), (352, 72, 24, 32), (1152, 1032, 16, 128)])
def test_packed(bits, i, o, r, g):
    from oracle import l4q_oracle as O
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"pack{bits}_{o}x{i}", 8, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=bits + i)
    s, b = host_qparams(spec, arrs, "asymm", 0.8)
    s[0, 0] = 2.0 ** -70  # one scale outside the reciprocal's range: its row block takes the IEEE divide
    layer = binding.upload(spec, arrs, s, b)
    got = packed_on_gpu(spec, layer).cpu().numpy().view(np.uint32)
    dec, _, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    assert np.array_equal(got, O.pack_codes(dec.codes, bits))


@pytest.mark.parametrize("method,mid", [("asymm", 0), ("symm", 1), ("l4q", 2)])
@pytest.mark.parametrize("i,o,g", [(96, 40, 32), (320, 8, 64), (640, 1032, 128), (768, 264, 256)])
def test_init(method, mid, i, o, g):
    import torch
    from oracle import l4q_oracle as O
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"init_{method}_{o}x{i}_g{g}", 8, i, o, 16, 24.0, 3, g, DTYPE_BF16)  # gamma = 1.5: no power of two
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=g)
    layer = binding.upload(spec, arrs)
    binding.l4q_init_qparams(layer.desc, layer.W0, layer.A, layer.B, mid, layer.scale, layer.zero)
    torch.cuda.synchronize()
    s, b = O.init_qparams(O.merge_f32(arrs["W0"], arrs["A"], arrs["B"], spec.alpha), 3, g, method, dtype=np.float32)
    assert np.array_equal(layer.scale.cpu().numpy().view(np.uint32), s.view(np.uint32))
    assert np.array_equal(layer.zero.cpu().numpy().view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("i,o,r,g,dtype", [
    (32, 8, 8, 32, DTYPE_BF16),         # four pairs, three of them of wavefronts past the last column
    (352, 1032, 8, 32, DTYPE_BF16),
    (1024, 72, 16, 1024, DTYPE_BF16),   # a group across strips
    (2560, 1000, 4, 64, DTYPE_BF16),    # the general pass: 10000 pairs, added in runs of 2048, the last one longer
    (512, 4097, 3, 64, DTYPE_F32),      # 8194 pairs: four runs
    (256, 2049, 3, 64, DTYPE_F32),      # 2049 pairs: one block
])
def test_error_sums(i, o, r, g, dtype):
    import torch
    from oracle import l4q_oracle as O
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"err_{o}x{i}_r{r}", 8, i, o, r, 2.0 * r, 4, g, dtype)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=i + o)
    s, b = host_qparams(spec, arrs, "asymm", 0.7)
    layer = binding.upload(spec, arrs, s, b)
    errors = torch.zeros(8, dtype=torch.float32, device=layer.W0.device)
    need = o * ((i + 255) // 256) * 8
    ws = torch.full((need + 256,), 0x7F, dtype=torch.uint8, device=layer.W0.device)
    binding.l4q_quant_errors(layer.desc, layer.W0, layer.A, layer.B, layer.scale, layer.zero, errors, ws[:need])
    binding.l4q_quant_errors_static(layer.desc, layer.W0, layer.A, layer.B, layer.scale, layer.zero, errors[4:])
    torch.cuda.synchronize()
    assert (ws[need:] == 0x7F).all()  # nothing past the stated size
    e = errors.cpu().numpy()
    Wc = O.merge(arrs["W0"], arrs["A"], arrs["B"], spec.alpha)
    want = np.array([O.quantization_error(Wc, s, b, 4, g), O.clipping_error(Wc, s, b, 4, g)])
    # binary32 terms of |Wc| <= 2 with 2^-24 rounding each and decisions a rounding away from a tie, whose two codes are
    # equally far: well below 1e-5 of sums that average a quarter of a step per weight
    assert np.allclose(e[:2], want, rtol=1e-5, atol=0), (e, want)
    assert np.array_equal(e[:2], e[4:6])


@pytest.mark.parametrize("what", ["weight", "zero", "both"])
@pytest.mark.parametrize("i,o,r,g", [(96, 40, 16, 32), (512, 72, 64, 128)])
def test_error_sums_beyond_the_quotients_range(i, o, r, g, what):
    """W / s or zero / s past the largest binary32 number, with the scale inside the reciprocal's range: the errors are
    finite, of the size of W or zero."""
    import torch
    from oracle import l4q_oracle as O
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"err_range_{what}_{o}x{i}_r{r}", 8, i, o, r, 2.0 * r, 4, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=i)
    s, b = host_qparams(spec, arrs, "asymm", 0.7)
    s[5, 1] = 2.0 ** -50
    W0 = np.asarray(arrs["W0"]).copy()
    if what != "zero":
        W0[5, g + 3], W0[5, g + 9] = 2.0 ** 100, -(2.0 ** 101)
    if what != "weight":
        b[5, 1] = 2.0 ** 100
    arrs["W0"] = W0
    layer = binding.upload(spec, arrs, s, b)
    errors = torch.zeros(4, dtype=torch.float32, device=layer.W0.device)
    ws = torch.zeros(o * ((i + 255) // 256) * 8, dtype=torch.uint8, device=layer.W0.device)
    binding.l4q_quant_errors(layer.desc, layer.W0, layer.A, layer.B, layer.scale, layer.zero, errors, ws)
    torch.cuda.synchronize()
    Wc = O.merge(arrs["W0"], arrs["A"], arrs["B"], spec.alpha)
    want = np.array([O.quantization_error(Wc, s, b, 4, g), O.clipping_error(Wc, s, b, 4, g)])
    assert np.allclose(errors[:2].cpu().numpy(), want, rtol=1e-5, atol=0), (errors, want)


@pytest.mark.parametrize("method", [0, 1, 2])
@pytest.mark.parametrize("i,o,g", [(96, 40, 32), (320, 40, 64), (768, 40, 256)])
def test_init_with_nan(method, i, o, g):
    """Rank 8 takes the streaming pass, rank 4 the general one: the same weight (B = 0) has to come out the same, bit for
    bit, also where a group is partly or wholly NaN."""
    import torch
    from paper_2402_04902_amd import binding
    out = []
    for r in (8, 4):
        spec = LayerSpec(f"init_nan_{o}x{i}_g{g}_r{r}", 8, i, o, r, 2.0 * r, 3, g, DTYPE_BF16)
        print("case", spec.name, method, flush=True)
        arrs = inputs.make_layer_inputs(LayerSpec("w", 8, i, o, 8, 16.0, 3, g, DTYPE_BF16), seed=g)
        layer = binding.upload(LayerSpec("w", 8, i, o, 8, 16.0, 3, g, DTYPE_BF16), arrs)
        layer.W0[3, :g] = float("nan")              # a whole group
        layer.W0[o - 1, g:2 * g - 1] = float("nan")  # all of a group but its last weight
        layer.W0[5, 7] = float("nan")
        layer.W0[9, 2] = float("inf")
        layer.W0[10, 1] = -float("inf")
        A = layer.A[:r].contiguous()
        B = torch.zeros((o, r), dtype=torch.bfloat16, device=A.device)
        scale, zero = torch.full_like(layer.scale, 7.0), torch.full_like(layer.zero, 7.0)
        binding.l4q_init_qparams(binding.make_desc(spec), layer.W0, A, B, method, scale, zero)
        torch.cuda.synchronize()
        out.append(torch.stack([scale, zero]).cpu())
    streamed, general = out
    assert torch.equal(torch.isnan(streamed), torch.isnan(general))
    assert torch.equal(torch.nan_to_num(streamed, nan=7.0), torch.nan_to_num(general, nan=7.0))
