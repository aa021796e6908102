"""Where the QAT-LoRA backward takes the scale and zero gradients in the weight-gradient product's epilogue (l4q::dw_groups_used)
and where from the stored gradient: the GPU cases of either, and sizes where both were measured.  Host code alone."""
import ctypes

import pytest

from paper_2402_04902_amd import binding
from plan_util import _LayerDims

EPILOGUE = [(1, 1056, 2056, 4, 32), (70, 1312, 1288, 3, 32), (33, 1088, 1032, 2, 64), (97, 640, 776, 4, 128), (64, 768, 776, 8, 256),
            (161, 1280, 776, 5, 256), (600, 2048, 520, 4, 32)]  # (600 tokens: dB in partial sums)
STORED = [(1, 32, 8, 4, 32), (70, 288, 264, 3, 32), (33, 320, 520, 2, 64), (97, 512, 256, 4, 128), (64, 768, 72, 8, 256),
          (40, 512, 136, 4, 512)]


def in_epilogue(T, i, o, bits, g):
    f = getattr(binding.load_library(), "_ZN3l4q14dw_groups_usedERKNS_9LayerDimsE")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.POINTER(_LayerDims)]
    q = float(1 << (bits - 1))
    return f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)))


@pytest.mark.parametrize("case", EPILOGUE + STORED)
def test_gpu_cases_take_the_form_they_name(case):
    assert in_epilogue(*case) == (case in EPILOGUE)


@pytest.mark.parametrize("T,i,o,g,epilogue", [   # us of a step, stored / epilogue
    (33, 256, 256, 32, False),      # 45.7 / 51.6
    (293, 544, 368, 32, False),     # 57.6 / 60.3
    (2079, 512, 608, 256, False),   # 146.1 / 150.1
    (2048, 4096, 4096, 128, True),  # 290 / 263
])
def test_the_faster_form(T, i, o, g, epilogue):
    assert in_epilogue(T, i, o, 4, g) == epilogue
