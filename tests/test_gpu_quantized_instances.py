"""Quantized forward: the instances of its kernels that no other GPU case reaches, one call each, most with a ragged last row tile,
a partial last token block and rows that end inside a macro; against binary64, with what is not finite in its place.  Which instance a
call takes, and that none is left out, is checked on the host (test_quantized_instances.py)."""
import pytest

from test_gpu_blocks import quantized_forward_against_binary64

pytestmark = pytest.mark.gpu

# (T, in, out, bits, group), an instance it is there for (plan_util.quantized_instances)
CASES = [
    ((31, 704, 856, 2, 64), ("blocks", 2, 64, 1, 2)),
    ((12, 320, 4344, 2, 64), ("blocks", 2, 64, 2, 1)),
    ((24, 320, 4136, 2, 64), ("blocks", 2, 64, 2, 2)),
    ((45, 832, 4296, 2, 64), ("blocks", 2, 64, 2, 3)),
    ((149, 320, 4296, 2, 64), ("blocks", 2, 64, 2, 4)),
    ((14, 320, 8344, 2, 64), ("blocks", 2, 64, 3, 1)),
    ((19, 320, 8248, 2, 64), ("blocks", 2, 64, 3, 2)),
    ((39, 576, 8552, 2, 64), ("blocks", 2, 64, 3, 3)),
    ((346, 320, 8552, 2, 64), ("blocks", 2, 64, 3, 4)),
    ((44, 2432, 264, 2, 128), ("blocks", 2, 128, 1, 3)),
    ((11, 640, 4152, 2, 128), ("blocks", 2, 128, 2, 1)),
    ((13, 640, 11896, 2, 128), ("blocks", 2, 128, 3, 1)),
    ((47, 640, 8680, 2, 128), ("blocks", 2, 128, 3, 3)),
    ((57, 4416, 136, 4, 64), ("blocks", 4, 64, 1, 4)),
    ((3, 320, 4184, 4, 64), ("blocks", 4, 64, 2, 1)),
    ((20, 320, 4120, 4, 64), ("blocks", 4, 64, 2, 2)),
    ((35, 960, 4376, 4, 64), ("blocks", 4, 64, 2, 3)),
    ((274, 320, 4376, 4, 64), ("blocks", 4, 64, 2, 4)),
    ((18, 320, 8648, 4, 64), ("blocks", 4, 64, 3, 2)),
    ((46, 320, 8696, 4, 64), ("blocks", 4, 64, 3, 3)),
    ((116, 320, 8312, 4, 64), ("blocks", 4, 64, 3, 4)),
    ((14, 640, 4280, 4, 128), ("blocks", 4, 128, 2, 1)),
    ((14, 1088, 4152, 8, 64), ("blocks", 8, 64, 2, 1)),
    ((22, 320, 4344, 8, 64), ("blocks", 8, 64, 2, 2)),
    ((41, 832, 4296, 8, 64), ("blocks", 8, 64, 2, 3)),
    ((54, 320, 4120, 8, 64), ("blocks", 8, 64, 2, 4)),
    ((6, 640, 8200, 8, 128), ("blocks", 8, 64, 3, 1)),
    ((2, 30720, 5080, 2, 2048), ("decode", 2, 2)),   # (two stages of activations are all that fits beside such rows)
    ((1, 640, 21192, 2, 128), ("decode", 2, 4)),
    ((1, 640, 952, 2, 128), ("decode", 2, 8)),
    ((2, 30464, 4776, 4, 256), ("decode", 4, 2)),
    ((1, 5760, 4712, 4, 128), ("decode", 4, 4)),
    ((2, 31744, 40, 8, 1024), ("decode", 8, 2)),
    ((6, 320, 4104, 8, 64), ("decode", 8, 4)),
    ((21, 26432, 24, 2, 64), ("general", 2, 1, False)),  # (tables of such rows do not fit beside the other forms' rings)
    ((19, 26688, 24, 4, 64), ("general", 4, 1, False)),
    ((2, 25792, 24, 8, 64), ("general", 8, 1, False)),
    ((23, 28160, 24, 4, 64), ("stream", 4, 32)),
    ((1, 16000, 40, 8, 64), ("stream", 8, 16)),
    ((1, 17152, 10408, 3, 256), ("tile", 3, 1, False)),
    ((1, 25088, 24, 3, 256), ("tile", 3, 1, True)),
    ((29, 768, 22232, 3, 128), ("tile", 3, 2, False)),
    ((277, 11520, 56, 3, 128), ("tile", 3, 2, True)),
    ((99, 8448, 72, 3, 256), ("tile", 3, 3, True)),
    ((260, 15104, 40, 3, 256), ("tile", 3, 4, True)),
    ((396, 25600, 24, 4, 256), ("tile", 4, 1, True)),
    ((21, 768, 21544, 4, 128), ("tile", 4, 2, False)),
    ((414, 25600, 24, 4, 1024), ("tile", 4, 2, True)),
    ((103, 3584, 168, 4, 128), ("tile", 4, 3, True)),
    ((3, 22528, 12680, 8, 2048), ("tile", 8, 1, False)),
    ((217, 15232, 40, 8, 128), ("tile", 8, 2, True)),
    ((234, 25472, 24, 8, 64), ("tile", 8, 3, True)),
    ((24, 384, 1576, 2, 128), ("wreg", 2, 1, 1, 8)),
    ((1, 4480, 2504, 2, 128), ("wreg", 2, 1, 2, 16)),
    ((1, 13952, 2136, 2, 128), ("wreg", 2, 1, 4, 16)),
    ((4, 640, 4184, 2, 128), ("wreg", 2, 2, 1, 16)),
    ((2, 5504, 4408, 2, 128), ("wreg", 2, 2, 2, 16)),
    ((4, 640, 12312, 2, 128), ("wreg", 2, 4, 1, 16)),
    ((22, 896, 728, 3, 128), ("wreg", 3, 1, 1, 8)),
    ((1, 6272, 104, 3, 128), ("wreg", 3, 1, 2, 16)),
    ((1, 16000, 56, 3, 128), ("wreg", 3, 1, 4, 16)),
    ((5, 640, 4344, 3, 128), ("wreg", 3, 2, 1, 16)),
    ((12, 640, 4200, 8, 128), ("wreg", 8, 2, 1, 16)),
]


@pytest.mark.parametrize("T,i,o,bits,g", [c[0] for c in CASES])
def test_instance(T, i, o, bits, g):
    quantized_forward_against_binary64(T, i, o, bits, g)
