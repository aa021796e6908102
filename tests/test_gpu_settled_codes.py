"""Codes that the forward and packing passes cannot take from their near sums: weights on rounding ties, alone, a few in a row
block of 32 rows x 64 columns, more of a lane (32 columns of a row) than are recomputed one by one, and everywhere; ranks with A
in registers and beyond; row blocks in turn with many, none, and no rank term; infinite factors.  Wq, Wq^T, the factor and
the packed words bit for bit against the oracle's binary32 chain."""
import numpy as np
import pytest

from oracle import l4q_oracle as O
from paper_2402_04902_amd import inputs
from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

from parity_util import check_workspace_state
from test_gpu_quantized_path import packed_on_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [1, 9, 60, 200, 2000, -1])
@pytest.mark.parametrize("i,o,r,g,bits", [(96, 40, 8, 32, 4), (320, 72, 16, 64, 3), (512, 136, 64, 128, 2), (256, 64, 72, 256, 8),
                                          (256, 64, 136, 128, 5), (352, 72, 24, 32, 7)])
def test_ties(i, o, r, g, bits, ties):
    import torch
    from paper_2402_04902_amd import binding
    spec = LayerSpec(f"ties{ties}_{o}x{i}_r{r}_b{bits}", 8, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=i + r + bits)
    rng = np.random.default_rng(i + ties)
    # scale a power of two, zero 0: a weight of (k + 1/2) s is a tie.  B A is tiny (it decides the side) or cancels in pairs.
    s = np.full((o, i // g), 2.0 ** -6, np.float32)
    b = np.zeros((o, i // g), np.float32)
    qp = 2 ** (bits - 1) - 1
    # |quotients| near 1/4 elsewhere
    W0 = ((rng.integers(-qp, qp + 1, (o, i)) + 0.25) * 2.0 ** -6).astype(np.float32)
    tie = ((rng.integers(-qp, qp + 1, (o, i)) - 0.5) * 2.0 ** -6).astype(np.float32)
    if ties < 0:
        W0 = tie
    else:  # `ties` of them among the first 32 x 64 weights
        at = rng.permutation(min(o, 32) * min(i, 64))[:ties]
        W0[at // min(i, 64), at % min(i, 64)] = tie[at // min(i, 64), at % min(i, 64)]
    arrs["W0"] = inputs.round_to_bf16(W0)
    B = np.asarray(arrs["B"]) * 2.0 ** -12
    B[:, 1::2] = np.where(rng.random(B[:, 1::2].shape) < 0.5, -B[:, ::2], B[:, 1::2])
    arrs["B"] = inputs.round_to_bf16(B.astype(np.float32))
    A = np.asarray(arrs["A"]).copy()
    A[1::2] = np.where(rng.random(A[1::2].shape) < 0.9, A[::2], A[1::2])
    arrs["A"] = inputs.round_to_bf16(A)
    layer = binding.upload(spec, arrs, s, b)
    dec, _, w32 = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    layer.forward()
    layer.backward()
    torch.cuda.synchronize()
    check_workspace_state(spec, layer, dec, w32, s, b, fused=r <= 32)  # (above: the factor has been overwritten)
    got = packed_on_gpu(spec, layer).cpu().numpy().view(np.uint32)
    assert np.array_equal(got, O.pack_codes(dec.codes, bits))


def test_row_blocks_in_turn():
    """A wavefront's run of five and six row blocks: after one with many undecided codes it goes straight to the stated sums for
    three, then back; blocks without a rank term (rows of B all zero) take their near sums as they are, ties included."""
    import torch
    from paper_2402_04902_amd import binding
    i, o, r, g, bits = 16384, 2048, 8, 128, 4
    spec = LayerSpec("turns", 8, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    arrs = inputs.make_layer_inputs(spec, seed=9)
    rng = np.random.default_rng(9)
    block = np.arange(o) // 32
    tie = rng.random((o, i)) < np.select([block % 7 == 0, block % 7 == 5], [0.5, 0.002], 0.0)[:, None]
    tie |= (block % 3 == 1)[:, None] & (rng.random((o, i)) < 0.5)  # (the blocks without a rank term)
    W0 = ((rng.integers(-7, 8, (o, i)) + np.where(tie, -0.5, 0.25)) * 2.0 ** -6).astype(np.float32)
    arrs["W0"] = inputs.round_to_bf16(W0)
    B = np.asarray(arrs["B"]) * 2.0 ** -12
    B[block % 3 == 1] = 0
    arrs["B"] = inputs.round_to_bf16(B.astype(np.float32))
    s, b = np.full((o, i // g), 2.0 ** -6, np.float32), np.zeros((o, i // g), np.float32)
    dec, _, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    layer = binding.upload(spec, arrs, s, b)
    packed = packed_on_gpu(spec, layer).cpu().numpy().view(np.uint32)
    for n in range(8):
        assert np.array_equal((packed >> np.uint32(4 * n)) & np.uint32(15), (dec.codes[:, n::8] + 8).astype(np.uint32)), n
    layer.forward()
    torch.cuda.synchronize()
    wq = layer.ws[: o * i * 2].view(torch.int16).reshape(i // 32, o, 32).permute(1, 0, 2).reshape(o, i).cpu().numpy().view(np.uint16)
    assert np.array_equal(wq, inputs.bf16_bits((dec.codes * np.float32(2.0 ** -6)).astype(np.float32)))


def test_infinite_factor():
    """An infinite element of A: the near sums of its column do not count, and its wavefront's row blocks are repeated."""
    import torch
    from paper_2402_04902_amd import binding
    i, o, r, g, bits = 256, 64, 16, 64, 4
    spec = LayerSpec("inf_a", 8, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    arrs = inputs.make_layer_inputs(spec, seed=5)
    A = np.asarray(arrs["A"]).copy()
    A[3, 70] = np.inf
    arrs["A"] = A
    s, b = np.full((o, i // g), 0.01, np.float32), np.full((o, i // g), 0.002, np.float32)
    layer = binding.upload(spec, arrs, s, b)
    with np.errstate(invalid="ignore"):
        dec, _, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    got = packed_on_gpu(spec, layer).cpu().numpy().view(np.uint32)
    torch.cuda.synchronize()
    assert np.array_equal(got, O.pack_codes(dec.codes, bits))


@pytest.mark.parametrize("where,value", [("A", np.inf), ("B", -np.inf), ("B", np.nan)])
@pytest.mark.parametrize("r", [8, 16, 24, 64])
def test_weights_beside_a_nonfinite_factor(r, where, value):
    """The weights whose sums are finite, in the row block of one whose sum is not: forward and packing."""
    import torch
    from paper_2402_04902_amd import binding
    i, o, g, bits = 256, 72, 64, 4
    spec = LayerSpec(f"beside_r{r}_{where}{value}", 8, i, o, r, 2.0 * r, bits, g, DTYPE_BF16)
    print("case", spec.name, flush=True)
    arrs = inputs.make_layer_inputs(spec, seed=r)
    v = np.asarray(arrs[where]).copy()
    v[3, 7] = value  # (a column of the weight, or a row)
    arrs[where] = v
    s, b = np.full((o, i // g), 0.01, np.float32), np.full((o, i // g), 0.002, np.float32)
    layer = binding.upload(spec, arrs, s, b)
    with np.errstate(invalid="ignore"):
        dec, Wc, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    finite = np.isfinite(Wc)
    assert finite.sum() >= o * i - max(o, i)
    got = O.unpack_codes(packed_on_gpu(spec, layer).cpu().numpy().view(np.uint32), bits, i)
    assert np.array_equal(got[finite], dec.codes[finite])
    layer.forward()
    torch.cuda.synchronize()
    wq = layer.ws[: o * i * 2].view(torch.int16).reshape(i // 32, o, 32).cpu().numpy().view(np.uint16)
    wq = np.ascontiguousarray(wq.transpose(1, 0, 2)).reshape(o, i)
    want = (dec.codes.astype(np.float64) * np.float64(s[0, 0]) + np.float64(b[0, 0])).astype(np.float32)
    assert np.array_equal(wq[finite], inputs.bf16_bits(inputs.round_to_bf16(want))[finite])
