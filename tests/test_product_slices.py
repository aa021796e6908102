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
    (1024, 4096, 11008, 2),    # (training step) 423 against 445: halves in slices, not one pass of quarters
    # ... and as before: small tiles in slices
    (64, 4096, 28672, 8),
    # weights that it holds: as before
    (512, 4096, 4096, 1),
    (320, 4096, 4096, 2),
    (100, 4096, 4096, 6),
])
def test_forward_slices(T, o, i, slices):
    assert forward_slices(T, o, i) == slices


def backward_slices(T, o, i, r):
    def total(tokens):
        return binding.l4q_workspace_bytes(binding.make_desc(LayerSpec("plan", tokens, i, o, r, 2.0 * r, 4, 64, DTYPE_BF16)))[1]
    rest = total(T) - total(8192)  # (a product of many tiles: one pass; the other arrays do not depend on the tokens)
    assert rest % (T * i * 4) == 0
    return max(1, rest // (T * i * 4))


@pytest.mark.parametrize("r", [16, 64])
@pytest.mark.parametrize("T,o,i,slices", [
    # dX after the weight-gradient kernel: full tiles in slices from smaller weights on.  (Training steps at rank 16, us)
    (768, 11008, 4096, 5),   # 405 against 430
    (768, 7168, 7168, 3),    # 452 against 480
    (1500, 11008, 3072, 3),  # 465 against 493
    (512, 4096, 4096, 1),    # as before
    (320, 4096, 4096, 2),
])
def test_backward_slices(T, o, i, slices, r):
    assert backward_slices(T, o, i, r) == slices
