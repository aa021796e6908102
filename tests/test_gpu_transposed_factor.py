"""B^T as the backward merge passes leave it: its values at ranks that are and are not whole 16-byte pieces, over one and several
column strips, in the streaming pass and the general one; and what it adds to the time of a pass."""
import statistics

import numpy as np
import pytest

from plan_util import gpu_us, merge_quant_transposed

pytestmark = pytest.mark.gpu


def operands(i, o, r, g):
    import torch
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(r)
    W0 = (torch.randn((o, i), generator=gen, device=dev) * 0.02).bfloat16()
    B = torch.randn((o, r), generator=gen, device=dev).bfloat16()
    s = torch.full((o, i // g), 0.01, device=dev)
    wqT = torch.empty((i, (o + 31) // 32 * 32), dtype=torch.bfloat16, device=dev)
    return W0, B, s, torch.zeros_like(s), wqT


@pytest.mark.parametrize("g", [32, 8])  # (groups of 8: the general pass)
@pytest.mark.parametrize("i,o,r", [(96, 40, 3), (96, 40, 8), (1152, 264, 16), (1152, 1032, 250), (608, 200, 256), (4096, 4096, 24)])
def test_values(i, o, r, g):
    import torch
    W0, B, s, z, wqT = operands(i, o, r, g)
    guard = 64
    for ld in (o, (o + 31) // 32 * 32):  # rows of their own length (QAT-LoRA), and padded with zeros
        room = torch.full((r * ld + guard,), 7.0, dtype=torch.bfloat16, device=B.device)
        bT = room[:r * ld].view(r, ld)
        merge_quant_transposed(W0, B, s, z, 4, g, wqT, bT)
        torch.cuda.synchronize()
        assert torch.equal(bT[:, :o], B.t()) and not bT[:, o:].any() and (room[r * ld:] == 7.0).all()


@pytest.mark.parametrize("g", [128, 16])
def test_time(g):
    """Rank 256 of an 11008 x 4096 weight: 5.6 MB beside the pass's 180.  (All of it left to one strip's workgroups: 3.8 times the
    pass alone.)"""
    import torch
    W0, B, s, z, wqT = operands(4096, 11008, 256, g)
    bT = torch.empty((256, 11008), dtype=torch.bfloat16, device=B.device)
    t = {"without": [], "with": []}
    for _ in range(7):
        for k in t:
            t[k].append(gpu_us(lambda: merge_quant_transposed(W0, B, s, z, 4, g, wqT, bT if k == "with" else None)))
    alone, both = statistics.median(t["without"]), statistics.median(t["with"])
    print(f"groups of {g}: {alone:.1f} us, with B^T {both:.1f} us")
    assert both < 1.5 * alone
    assert np.array_equal(bT[:, 5].float().cpu().numpy(), B[5].float().cpu().numpy())
