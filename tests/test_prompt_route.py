"""Where a quantized forward of more than 64 tokens takes the two-dimensional tiles and where the passes of 64 tokens, at sizes
where both were measured (us, passes / tiles)."""
import pytest

from plan_util import PASSES, TILES_64x128, TILES_128x256, prompt_form, wide_tile_rows
from test_gpu_prefill import CASES


@pytest.mark.parametrize("T,o,i,bits,g", [
    (65, 8192, 11008, 2, 64),    # 88 / 107
    (65, 8192, 8192, 4, 64),     # 72 / 79
    (96, 8192, 8192, 3, 256),    # 60 / 72
    (256, 2048, 8192, 3, 256),   # 61 / 71
    (192, 4096, 8192, 4, 256),   # 59 / 64
    (64, 4096, 4096, 4, 128),    # not a prompt
    (300, 4096, 4096, 3, 64),    # no tiles for 3 bits in groups of 64
])
def test_passes(T, o, i, bits, g):
    assert prompt_form(T, i, o, bits, g) == PASSES


@pytest.mark.parametrize("T,o,i,bits,g,form", [
    (65, 11008, 4096, 4, 128, TILES_64x128),    # 44 / 32
    (129, 4096, 4096, 4, 128, TILES_64x128),    # 40 / 32
    (128, 8192, 11008, 4, 64, TILES_64x128),    # 123 / 105
    (300, 4096, 11008, 4, 128, TILES_64x128),   # 125 / 83
    (512, 11008, 4096, 4, 128, TILES_128x256),  # 215 / 66
])
def test_tiles(T, o, i, bits, g, form):
    assert prompt_form(T, i, o, bits, g) == form


@pytest.mark.parametrize("case,forms", CASES)
def test_gpu_cases_take_the_shapes_they_name(case, forms):
    T, i, o, g = case
    assert tuple(prompt_form(T, i, o, bits, g, False) for bits in (2, 3, 4, 8)) == forms


@pytest.mark.parametrize("T,i,o,bits,g", [(80, 2304, 4104, 8, 128), (100, 3072, 2048, 3, 512), (100, 3072, 2048, 4, 256)])
def test_two_pass_cases_of_the_quantized_path_are_passes(T, i, o, bits, g):
    assert prompt_form(T, i, o, bits, g, True) == PASSES


@pytest.mark.parametrize("T,o,rows", [
    (512, 11008, 192),   # 172 tiles of 256 rows, 232 of 192: one round either way
    (641, 8200, 256),    # 198 and 258: a second round
    (513, 7496, 192),
    (512, 16384, 256),   # 256 and 344
])
def test_wide_tile_rows(T, o, rows):
    assert wide_tile_rows(T, 4096, o, 4, 128) == rows
