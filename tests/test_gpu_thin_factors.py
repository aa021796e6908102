"""dA of ranks over 32: the thin product B^T . dWm with 64, 128 or 256 of a tile's columns multiplied, ranks on either side of those
lines, in-features that end inside a wave's columns, one stage to several slices of out-features, against the oracle."""
import pytest

from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [40, 64, 72, 128, 136])
@pytest.mark.parametrize("T,i,o", [(70, 352, 32), (33, 832, 1112)])
def test_thin_factors(r, T, i, o):
    run_case(LayerSpec(f"thin_{T}x{i}x{o}", T, i, o, r, 2.0 * r, 4, 32, DTYPE_BF16, outliers=False), seed=r, shrink=0.8)
