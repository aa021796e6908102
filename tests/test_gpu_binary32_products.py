"""Binary32 layers at the edges of the product kernels' forms (few tiles: k-slices over a workgroup's waves; 64-wide;
128-wide tiles): odd token and out-feature counts end tiles and k-steps everywhere, against the fp64 oracle."""
import pytest

from paper_2402_04902_amd.inputs import DTYPE_F32, LayerSpec

from test_gpu_parity import run_case
from test_gpu_qatlora import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,i,o,r,g", [
    (1, 4, 1, 1, 4),            # one element of everything
    (33, 36, 31, 5, 4),         # sliced form, k tails shorter than a run of 8
    (7, 260, 129, 8, 4),        # sliced form, K = 7 and K = 129
    (1037, 1028, 1031, 3, 4),   # 64-wide tiles in the forward product, dX and dWq; K = 1031, 1037
    (16, 2052, 2051, 2, 4),     # 64-wide tiles on one k-step of 16 (dWq)
    (1057, 1060, 1025, 3, 4),   # 64-wide tiles, the k-steps dealt to two groups of waves: the last one to the first
    (129, 2052, 2051, 2, 4),    # ... five steps, the last of one row (dWq)
    (35, 2948, 2949, 2, 4),     # 128-wide tiles (dWq: 24 x 24, both operands K-major), K = 35
    (2945, 36, 2945, 2, 4),     # ... in the forward product (24 x 24, both K-contiguous), K = 36
    (2945, 2948, 35, 2, 4),     # ... in dX (24 x 24, one of each), K = 35
    # operands of whole 16-byte pieces, straight to LDS:
    (1037, 1028, 1028, 3, 4),   # 64-wide tiles, ragged everywhere, K = 1028 (33 steps, the last of 4) and 1037 (of 13)
    (1025, 1088, 1056, 3, 4),   # whole steps, an even and an odd number of them; K = 1025: the last step of one row
    (2945, 2948, 36, 2, 4),     # 128-wide tiles in dX (one operand of each kind), K = 36
    (132, 2948, 2948, 2, 4),    # ... in dWq (both K-major, 2948 = 23 tiles and 4 columns), K = 132
    (2945, 260, 2948, 2, 4),    # ... in the forward product (both K-contiguous), K = 260
])
def test_binary32_product_forms(T, i, o, r, g):
    run_case(LayerSpec(f"f32_prod_{T}x{i}x{o}", T, i, o, r, 2.0 * r, 4, g, DTYPE_F32), seed=T + i, shrink=0.8)


@pytest.mark.parametrize("T,i,o,r", [
    (1037, 1028, 1031, 37),   # the rank term added to Y and dX in 64-wide tiles (17 x 17), one group of waves
    (1037, 1028, 1031, 150),  # ... two groups, five k-steps
    (2945, 36, 2945, 5),      # ... to Y in 128-wide tiles
    (2945, 2948, 35, 5),      # ... to dX
])
def test_binary32_rank_terms(T, i, o, r):
    _run(LayerSpec(f"f32_rank_{T}x{i}x{o}_r{r}", T, i, o, r, 2.0 * r, 4, 4, DTYPE_F32, outliers=False), seed=T + r)
