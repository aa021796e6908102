"""The quantized forward's GPU cases and the instances of its kernels (l4q::qgemm_route): every case runs the one it is there for, and
every instance that calls reach is run by a case, with what the query tells as workspace or without.  Host code alone (256 compute
units are assumed)."""
import random

import pytest

import test_blocks_route
import test_gpu_prefill
import test_gpu_quantized_instances
import test_gpu_quantized_path as path
from plan_util import quantized_instances, workspace_bytes


def instances(case):
    return set().union(*(quantized_instances(*case, w) for w in {False, workspace_bytes(*case) > 0}))


@pytest.mark.parametrize("case,instance", test_gpu_quantized_instances.CASES)
def test_gpu_cases_run_the_instances_they_name(case, instance):
    assert instance in instances(case)


def parameters(test):
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize")


def gpu_cases():
    cases = [c for c, _ in test_gpu_quantized_instances.CASES + test_blocks_route.GPU_CASES + test_blocks_route.GPU_PASSES]
    for draw in (path._random_forward_cases, path._random_tile_cases, path._random_in_register_cases):
        cases += [c[1:] for c in draw()]
    cases += parameters(path.test_quantized_forward_weights_in_registers)
    cases += parameters(path.test_quantized_forward_matches_oracle_and_training_forward)
    return cases + [(T, i, o, bits, g) for (T, i, o, g), _ in test_gpu_prefill.CASES for bits in (2, 3, 4, 8)]


def drawn_calls(count, rng):
    """Of every code width and group size, rows and tokens over the whole range, within the entry point's limits."""
    while count > 0:
        bits, g = rng.choice([2, 3, 4, 8]), 8 << rng.choice([0, 1, 2, 3, 3, 3, 3, 4, 4, 4, 4, 5, 5, 6, 7, 8, 9])
        unit = max(g, 64)
        i, o = unit * max(1, round((32768 / unit) ** rng.random())), 8 * round(3600 ** rng.random())
        T = rng.choice([rng.randint(1, 16), rng.randint(1, 64), rng.randint(1, 64), rng.randint(65, 600)])
        if max(T * i, T * o, o * (i + 64), i * (o + 64)) < 535_000_000:
            count -= 1
            yield T, i, o, bits, g


def test_every_instance_is_run_by_a_gpu_case():
    run = set().union(*map(instances, gpu_cases()))
    assert len(run) >= 155
    for case in drawn_calls(40000, random.Random(4902)):
        assert instances(case) <= run, case
