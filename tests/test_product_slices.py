"""Which products of the bfloat16 layer go in k-slices, as far as the stated workspace shows it: the padded weight and, per
slice, one binary32 tile of the output.  (Without a GPU the library plans for 256 compute units.)"""
import pytest

from paper_2402_04902_amd import binding
from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec


def forward_slices(T, o, i):
    desc = binding.make_desc(LayerSpec("plan", T, i, o, 16, 32.0, 4, 64, DTYPE_BF16))
    fwd, _ = binding.l4q_workspace_bytes(desc)
    assert i % 32 == 0 and (T * o * 4) % 256 == 0 and (o * i * 2) % 256 == 0
    rest = fwd - o * i * 2
    assert rest % (T * o * 4) == 0
    return max(1, rest // (T * o * 4))


@pytest.mark.parametrize("T,o,i,slices", [
    # weights that the cache does not hold: full tiles in slices, not one pass of small ones.  (Times with the merge pass, us)
    (512, 9600, 9600, 3),      # 190 against 237
    (256, 11008, 11008, 5),    # 191 against 234
    (640, 7168, 11008, 3),     # 183 against 212
    (1024, 5120, 13824, 3),    # 210 against 244
    (512, 8192, 11008, 4),     # 182 against 200
    (512, 8192, 14336, 4),     # 235 against 263
    # ... and as before: small tiles in slices
    (64, 4096, 28672, 8),
    # weights that it holds: as before
    (512, 4096, 4096, 1),
    (1024, 4096, 11008, 1),
    (320, 4096, 4096, 2),
    (100, 4096, 4096, 6),
])
def test_forward_slices(T, o, i, slices):
    assert forward_slices(T, o, i) == slices
