"""Time of the transposed rank products of few rows (one launch) by the layout of their result."""
import statistics

import pytest

from plan_util import gpu_us, transposed_rank_product

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n", [(16, 1024), (128, 2048)])
def test_layouts_take_the_same_time(T, n):
    """[n, r] against [r, n], rank 256.  (With the lanes of a store on consecutive ranks, whose sums lie in one bank: 1.3 times.)"""
    import torch
    r, dev = 256, torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(T)
    U, Xs = torch.randn((T, r), generator=gen, device=dev), torch.randn((T, n), generator=gen, device=dev)
    partial = torch.empty((2, r, n), device=dev)
    outs = {False: torch.empty((r, n), device=dev), True: torch.empty((n, r), device=dev)}
    t = {k: [] for k in outs}
    for _ in range(9):
        for k in t:
            t[k].append(gpu_us(lambda: transposed_rank_product(U, Xs, k, partial, outs[k])))
    rn, nr = statistics.median(t[False]), statistics.median(t[True])
    print(f"{T} rows: [r, n] {rn:.1f} us, [n, r] {nr:.1f} us")
    assert torch.equal(outs[False], outs[True].t())
    assert nr < 1.15 * rn


def test_two_row_blocks_of_a_high_rank():
    """[n, r]: 200 rows against 128, twice the partial sums and a second launch.  (Both row blocks in one workgroup: 1.7 times.)"""
    import torch
    r, n, dev = 256, 1024, torch.device("cuda:0")
    partial, out = torch.empty((2, r, n), device=dev), torch.empty((n, r), device=dev)
    args = {T: (torch.randn((T, r), device=dev), torch.randn((T, n), device=dev)) for T in (128, 200)}
    t = {T: [] for T in args}
    for _ in range(9):
        for T in t:
            t[T].append(gpu_us(lambda: transposed_rank_product(*args[T], True, partial, out)))
    one, two = statistics.median(t[128]), statistics.median(t[200])
    print(f"128 rows {one:.1f} us, 200 rows {two:.1f} us")
    assert two < 1.35 * one
