"""How a quantized forward of up to 64 tokens goes through the one-pass kernel (l4q::qgemm_blocks_plan): row tiles per workgroup
and k-slices, at sizes where the choice was measured, and that the GPU cases cover the forms they name.  Host code alone (256
compute units are assumed)."""
import ctypes
import timeit

import pytest

from paper_2402_04902_amd import binding
from plan_util import _BlocksPlan, _LayerDims, prompt_plan, workspace_bytes
from test_gpu_prefill import CASES

NOT_THIS_FORM = (0, 1)


def blocks_plan(T, i, o, bits, g, workspace=None):  # None: as given what the query tells
    if workspace is None:
        workspace = workspace_bytes(T, i, o, bits, g) > 0
    f = getattr(binding.load_library(), "_ZN3l4q17qgemm_blocks_planERKNS_9LayerDimsEb")
    f.restype, f.argtypes = _BlocksPlan, [ctypes.POINTER(_LayerDims), ctypes.c_bool]
    q = float(1 << (bits - 1))
    return f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)), workspace)


def blocks_form(*call):
    p = blocks_plan(*call)
    return p.nt, p.slices


# (T, in, out, bits, group), (tiles per workgroup, slices): every count of tiles and token blocks, k-slices, each code width in
# groups of 64 and more; rows of one step to many macros that do not divide among the waves, the last one partial; ragged tiles
GPU_CASES = [
    ((33, 128, 40, 4, 128), (1, 1)),      # one code step, seven idle waves
    ((48, 64, 24, 8, 64), (1, 1)),        # half a load of codes
    ((5, 320, 72, 2, 64), (1, 1)),
    ((16, 2176, 4104, 3, 128), (2, 1)),   # 257 tiles
    ((9, 1600, 9000, 4, 64), (3, 1)),
    ((33, 192, 88, 4, 64), (1, 1)),
    ((32, 4352, 2600, 3, 256), (1, 1)),   # 17 macros: three for one wave, two for the others
    ((31, 2368, 8200, 8, 64), (3, 1)),
    ((40, 640, 6008, 2, 128), (2, 1)),
    ((48, 4480, 11000, 4, 128), (3, 1)),
    ((47, 8704, 520, 4, 512), (1, 4)),   # slices that divide groups
    ((64, 4352, 4000, 4, 128), (1, 1)),
    ((64, 8704, 2600, 4, 128), (2, 3)),
    ((48, 11008, 4352, 3, 128), (3, 2)),
    ((50, 4224, 4096, 2, 128), (1, 1)),
    ((64, 1088, 10000, 8, 64), (3, 1)),
    ((64, 3072, 9000, 3, 128), (3, 1)),
    ((63, 8192, 264, 8, 64), (1, 4)),
]


@pytest.mark.parametrize("case,form", GPU_CASES)
def test_gpu_cases_take_the_forms_they_name(case, form):
    assert blocks_form(*case) == form


@pytest.mark.parametrize("T,i,o,bits,g", [
    (1, 4096, 11008, 4, 128),    # 8.0 in registers / 9.9
    (8, 4096, 11008, 4, 128),    # 9.2 / 9.7
    (2, 6144, 5120, 3, 128),     # the codes are all there is to load
    (24, 1024, 11008, 3, 128),   # 7.5 / 8.1
    (17, 4096, 14336, 4, 128),   # 15.7 / 17.1
    (43, 4096, 4096, 3, 64),     # no 3 bits in groups of 64
    (43, 4096, 4096, 4, 32),     # groups below 64
    (65, 4096, 4096, 4, 128),    # more than four blocks
    # short rows, a tile per unit: activations in LDS (us in a graph, that kernel / this one)
    (4, 512, 512, 4, 128),       # 3.7 / 4.0
    (12, 1024, 4096, 4, 256),    # 4.0 / 4.2
    (2, 3072, 2048, 4, 128),     # 4.7 / 5.1
    (2, 5120, 2048, 4, 128),     # 5.4 / 5.8
    (3, 512, 2048, 8, 64),       # 3.6 / 4.4
    (16, 1024, 512, 8, 128),     # 4.3 / 4.6
    (6, 2560, 1000, 8, 128),     # 5.0 / 5.4
    (16, 384, 8192, 8, 64),      # 4.4 / 5.6
    # two chunks per wave in registers
    (3, 8192, 8192, 3, 128),     # 11.3 / 11.9
    (7, 7424, 6144, 2, 128),     # 0.95 times
    # two token blocks in registers, the streaming form, 64-row tiles
    (17, 512, 3944, 3, 256),     # 4.7 / 5.1
    (20, 512, 1000, 2, 128),
    (17, 128, 8848, 8, 128),     # 5.2 / 6.6
    (32, 256, 12000, 4, 64),     # 6.0 / 6.9
    (50, 256, 11808, 8, 256),    # 6.1 / 10.1
    (64, 1024, 11280, 8, 256),   # 11.2 / 12.7
])
def test_other_kernels(T, i, o, bits, g):
    assert blocks_form(T, i, o, bits, g) == NOT_THIS_FORM


@pytest.mark.parametrize("T,i,o,bits,g", [
    # ... and beside those
    (13, 1024, 4096, 4, 256), (5, 3072, 2048, 4, 128), (3, 5120, 2048, 4, 128), (2, 2048, 2048, 4, 128), (7, 2560, 1000, 8, 128),
    (3, 512, 2048, 8, 128), (17, 1024, 8192, 8, 64), (8, 8192, 8192, 3, 128), (33, 512, 3944, 3, 256), (17, 1152, 3944, 3, 128),
    (33, 256, 12000, 4, 64), (33, 128, 8000, 8, 128), (50, 256, 10000, 8, 256), (48, 1024, 11280, 8, 256),
])
def test_this_kernel_beside_other_kernels(T, i, o, bits, g):
    assert blocks_form(T, i, o, bits, g) != NOT_THIS_FORM


def passes(T, i, o, bits, g, workspace=None):
    return planned_passes(T, i, o, bits, g, workspace)()


def planned_passes(T, i, o, bits, g, workspace=None):
    if workspace is None:
        workspace = workspace_bytes(T, i, o, bits, g) > 0
    f = getattr(binding.load_library(), "_ZN3l4q19qgemm_blocks_passesERKNS_9LayerDimsEbdPNS_10BlocksPlanE")
    f.restype, f.argtypes = ctypes.c_int, [ctypes.POINTER(_LayerDims), ctypes.c_bool, ctypes.c_double, ctypes.POINTER(_BlocksPlan)]
    q = float(1 << (bits - 1))
    dims, plans = _LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False), (_BlocksPlan * 8)()
    other_us = prompt_plan(T, i, o, bits, g, workspace).us
    return lambda: f(ctypes.byref(dims), workspace, other_us, plans)


# more than 64 tokens: the number of passes
GPU_PASSES = [
    ((65, 4096, 520, 4, 128), 2),     # of 32 and 33 tokens
    ((97, 4160, 1000, 2, 64), 2),
    ((150, 8192, 1040, 8, 128), 3),   # with room for partial sums, slices in each
    ((250, 8192, 1024, 4, 128), 4),
]


@pytest.mark.parametrize("case,n", GPU_PASSES)
def test_gpu_cases_take_the_passes_they_name(case, n):
    assert passes(*case) == n


@pytest.mark.parametrize("T,i,o,bits,g,n", [
    (64, 4096, 4096, 4, 128, 0),      # not more than 64 tokens
    (128, 4096, 4096, 4, 128, 2),     # 17.1 against 28.9 in two-dimensional tiles
    (256, 4096, 4096, 4, 128, 0),
    (65, 11008, 4096, 4, 128, 2),     # 28.4 / 40.5
    (128, 4096, 11008, 4, 128, 0),    # 32.4 / 29.6
    (65, 11008, 1024, 2, 128, 2),     # 24.6 / 78.4 in the general kernel's passes
    (256, 8192, 1024, 4, 128, 4),     # 36.8 / 50.9
    (512, 4096, 11008, 4, 128, 0),
    (600, 4096, 4096, 4, 128, 0),
])
def test_passes(T, i, o, bits, g, n):
    assert passes(T, i, o, bits, g) == n


def test_passes_of_the_same_size_are_planned_once():
    """Host time of the plan for eight passes of 64 tokens against one pass: the loop's own steps, not eight plans (5 to 6 times)."""
    def us(call):
        return min(timeit.repeat(call, number=300, repeat=15))
    eight, one = planned_passes(512, 16384, 256, 2, 64), planned_passes(65, 16384, 256, 2, 64)  # (65: two plans)
    assert eight() == 8 and one() == 2
    assert us(eight) <= 1.5 * us(one)


@pytest.mark.parametrize("case,forms", CASES)
def test_the_prompt_kernels_gpu_cases_are_not_taken_from_it(case, forms):
    T, i, o, g = case
    assert not any(passes(T, i, o, bits, g, False) for bits in (2, 3, 4, 8))


def test_slices_only_with_a_workspace():
    assert blocks_form(48, 11008, 4352, 3, 128)[1] == 2
    assert blocks_form(48, 11008, 4352, 3, 128, False)[1] == 1


def test_short_calls_have_one_launch():
    assert blocks_form(8, 8192, 1024, 4, 128)[1] == 1   # eager 7.9 us, in two launches 10.2
    assert blocks_form(3, 4224, 232, 8, 64)[1] == 1     # 7.9 / 10.2
    assert blocks_form(16, 11008, 1024, 4, 64)[1] > 1


@pytest.mark.parametrize("i", [1024, 4096, 5120, 11264, 16384])
@pytest.mark.parametrize("bits,g", [(2, 64), (3, 128), (4, 128), (4, 1024), (8, 64)])
def test_the_workspace_that_is_told_has_room_for_every_plans_slices(i, bits, g):
    for o in (8, 264, 1328, 2048, 3000, 4096, 6008, 11008):
        told = [workspace_bytes(T, i, o, bits, g) for T in (1, 53, 64, 300)]
        assert len(set(told)) == 1  # (it does not depend on the tokens)
        for T in (2, 5, 16, 17, 33, 53, 64):
            slices = blocks_plan(T, i, o, bits, g, True).slices
            assert slices == 1 or slices * T * o * 4 <= told[0]


@pytest.mark.parametrize("T,i,o,bits,g,slices", [
    (53, 10816, 1328, 2, 64, 3),   # 11.8 us (estimated) against 19.5 in one slice
    (17, 8192, 264, 8, 64, 4),
])
def test_a_caller_with_the_workspace_that_is_told_gets_the_slices(T, i, o, bits, g, slices):
    assert blocks_form(T, i, o, bits, g)[1] == slices


@pytest.mark.parametrize("T", [16, 63, 64])
@pytest.mark.parametrize("bits,g", [(2, 64), (3, 128), (4, 128), (8, 64)])
@pytest.mark.parametrize("i", [3072, 4096, 11008])
def test_room_for_partial_sums_never_makes_the_plan_slower(T, i, bits, g):
    for o in range(1032, 8200, 184):
        assert blocks_plan(T, i, o, bits, g, True).us <= blocks_plan(T, i, o, bits, g, False).us


@pytest.mark.parametrize("T", [128, 160, 176, 192, 256])
def test_passes_do_not_depend_on_room_where_one_slice_is_the_faster_plan(T):
    assert passes(T, 4096, 4096, 4, 128) == passes(T, 4096, 4096, 4, 128, False)
