"""The library's internal choice of kernel for a call, asked of the host code alone (no GPU: 256 compute units are assumed)."""
import ctypes

from paper_2402_04902_amd import binding


class _LayerDims(ctypes.Structure):  # LayerDims of csrc/l4q_kernels.h
    _fields_ = [("T", ctypes.c_int64), ("i", ctypes.c_int64), ("o", ctypes.c_int64), ("r", ctypes.c_int), ("bits", ctypes.c_int),
                ("g", ctypes.c_int), ("gamma", ctypes.c_float), ("qn", ctypes.c_float), ("qp", ctypes.c_float),
                ("accumulate", ctypes.c_bool)]


class _PrefillPlan(ctypes.Structure):
    _fields_ = [("form", ctypes.c_int), ("us", ctypes.c_double)]


PASSES, TILES_64x128, TILES_128x128, TILES_128x256 = -1, 0, 1, 2


def prompt_form(T, i, o, bits, g, workspace=True):
    """l4q::qgemm_prompt_plan: the tile shape a quantized forward of more than 64 tokens takes, or PASSES."""
    f = getattr(binding.load_library(), "_ZN3l4q17qgemm_prompt_planERKNS_9LayerDimsEb")
    f.restype, f.argtypes = _PrefillPlan, [ctypes.POINTER(_LayerDims), ctypes.c_bool]
    q = float(1 << (bits - 1))
    return f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)), workspace).form


def wide_tile_rows(T, i, o, bits, g):
    """l4q::qgemm_prompt_wide_rows: the weight rows of a 128-token wide tile for this call (what TILES_128x256 stands for)."""
    f = getattr(binding.load_library(), "_ZN3l4q22qgemm_prompt_wide_rowsERKNS_9LayerDimsE")
    f.restype, f.argtypes = ctypes.c_int, [ctypes.POINTER(_LayerDims)]
    q = float(1 << (bits - 1))
    return f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)))
