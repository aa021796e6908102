"""Rows per wave and per workgroup of the binary32 merge and quantizer-gradient passes, by layer size: every form, heights
that end inside a workgroup, widths that end inside a 256-column unit; bfloat16 layers through the unfused backward."""
import numpy as np
import pytest

from paper_2402_04902_amd import inputs
from paper_2402_04902_amd.inputs import DTYPE_BF16, DTYPE_F32, LayerSpec

from parity_util import check_float_outputs, host_qparams, oracle_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("i,o,r,g", [
    (64, 1, 1, 16),
    (264, 511, 17, 8),     # 1 row per wave and per workgroup; a second dB pass of one rank
    (320, 515, 16, 64),    # 2 rows per workgroup, the last one half filled
    (1280, 777, 5, 128),   # 2 rows per wave
    (512, 1030, 33, 512),  # groups longer than a unit
])
def test_layer(i, o, r, g):
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"rows_{o}x{i}_r{r}", 40, i, o, r, 2.0 * r, 3, g, DTYPE_F32)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=o)
    s, b = host_qparams(spec, arrs, "asymm", 0.7)
    layer = binding.upload(spec, arrs, s, b)
    layer.forward()
    layer.backward()
    _, _, _, Y, gr = oracle_all(spec, arrs, s, b)
    check_float_outputs(spec, layer, Y, gr)


def test_merge_of_a_layer_larger_than_one_resident_round():
    """4 rows per wave: codes read back through one-hot tokens, whose products are single entries of Wq."""
    import torch
    from oracle import l4q_oracle as O
    from paper_2402_04902_amd import binding
    i, o, r, g = 4096, 1101, 3, 64  # 16 x 69 workgroups at 2 rows per wave
    spec = LayerSpec("rows_4", 64, i, o, r, 6.0, 4, g, DTYPE_F32)
    arrs = inputs.make_layer_inputs(spec, seed=3)
    cols = np.linspace(0, i - 1, 64).astype(int)
    X = np.zeros((64, i), np.float32)
    X[np.arange(64), cols] = 1.0
    arrs["X"] = X
    s, b = host_qparams(spec, arrs, "asymm", 0.8)
    layer = binding.upload(spec, arrs, s, b)
    layer.forward()
    torch.cuda.synchronize()
    dec, _, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, 4, g, spec.alpha)
    Y = layer.Y.double().cpu().numpy()
    sc, bc = s[:, cols // g].astype(np.float64), b[:, cols // g].astype(np.float64)
    assert np.array_equal(np.rint((Y.T - bc) / sc), dec.codes[:, cols])


@pytest.mark.parametrize("i,o,r", [(256, 72, 9), (320, 1032, 20)])
def test_unfused_bf16(i, o, r):
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"unfused_{o}x{i}_r{r}", 40, i, o, r, 2.0 * r, 4, 64, DTYPE_BF16)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=o)
    s, b = host_qparams(spec, arrs, "asymm", 0.7)
    layer = binding.upload(spec, arrs, s, b, flags=binding.FLAG_UNFUSED_BACKWARD)
    layer.forward()
    layer.backward()
    _, _, _, Y, gr = oracle_all(spec, arrs, s, b)
    check_float_outputs(spec, layer, Y, gr)
