"""The sums of a split dX product and of the partial dA and dB in one launch: arrays that end inside a workgroup's share on either
side, both forms of the weight-gradient kernel, adding to the caller's gradients, against the oracle."""
import pytest

from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

from test_gpu_parity import run_case
from test_product_slices import backward_slices

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,i,o,r", [
    (37, 1088, 2056, 8),    # 39.3 workgroups of dX, 34 of dA, 64.25 of dB
    (130, 1088, 2056, 12),  # three quarters of a tile of ranks
    (1, 320, 4104, 4),      # 80 quads of dX: less than one workgroup
    (65, 1600, 2056, 36),   # the masked gradient's products, in slices of their own
])
def test_shared_sums(T, i, o, r):
    import torch
    from paper_2402_04902_amd import binding
    assert backward_slices(T, o, i, r) > 1
    _, layer, _ = run_case(LayerSpec(f"sums_{T}x{i}x{o}", T, i, o, r, 2.0 * r, 4, 64, DTYPE_BF16, outliers=False), seed=T, shrink=0.8)
    once = [g.clone() for g in (layer.dA, layer.dB, layer.dX)]
    layer.desc.flags = binding.FLAG_ACCUMULATE_GRADS
    layer.backward()
    torch.cuda.synchronize()
    assert torch.equal(layer.dA, 2 * once[0]) and torch.equal(layer.dB, 2 * once[1])  # (x + x is exact)
    assert torch.equal(layer.dX, once[2])
