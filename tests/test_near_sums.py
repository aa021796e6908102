"""The bound between the streaming pass's near rank sums (bfloat16 matrix ops) and the stated ones, on which its codes rest:
the matrix op's own error against exact sums, and codes that only that bound keeps right."""
import numpy as np
import pytest

from oracle import l4q_oracle as O
from paper_2402_04902_amd import inputs
from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec

U = 2.0 ** -24


# ---- the sums themselves.  W0 = 0, gamma = 1, zero = 0, one column of A and one row of B: the error sum of the layer, formed
# from near values, is |near sum| exactly when the scale is a power of two above four times it (its code is then 0).
def factors(kind, r, n, rng):
    """n pairs of factor vectors [n, r]"""
    if kind in ("cut", "after"):
        # products 0.99 of a power of two, 18 to 30 binary places below one large product: first (so that it comes back from the
        # accumulator for the later ops), or anywhere in the first op
        A = np.full((n, r), 1.9921875)
        B = A * 2.0 ** rng.integers(-30, -17, (n, 1)) * rng.choice([1.0, -1.0], (n, 1))
        at = np.zeros(n, int) if kind == "after" else rng.integers(0, min(r, 16), n)
        if kind == "after":
            A[:, 1:16] = 0
        big = rng.choice([1.0, 1.9921875], (2, n))
        A[np.arange(n), at], B[np.arange(n), at] = big
    else:
        spread = {"near": 3, "spread": 12, "far": 60}[kind]
        A = rng.normal(size=(n, r)) * 2.0 ** rng.integers(0, spread // 2 + 1, (n, r))
        B = rng.normal(size=(n, r)) * 2.0 ** rng.integers(0, spread // 2 + 1, (n, r))
    return inputs.round_to_bf16(A.astype(np.float32)), inputs.round_to_bf16(B.astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["cut", "after", "near", "spread", "far"])
@pytest.mark.parametrize("r", [8, 16, 24, 64, 72, 256])
def test_matrix_op_sums(r, kind):
    import torch
    from paper_2402_04902_amd import binding
    n, i, o, dev = 256, 32, 8, "cuda:0"
    Ak, Bk = factors(kind, r, n, np.random.default_rng(r))
    exact = (Ak.astype(np.float64) * Bk.astype(np.float64)).sum(1)
    S = np.abs(Ak.astype(np.float64) * Bk.astype(np.float64)).sum(1)
    desc = binding.make_desc(LayerSpec("near", 8, i, o, r, float(r), 4, 32, DTYPE_BF16))
    A, B = torch.zeros((n, r, i), device=dev), torch.zeros((n, o, r), device=dev)
    A[:, :, 5], B[:, 3] = torch.from_numpy(Ak).to(dev), torch.from_numpy(Bk).to(dev)
    A, B = A.bfloat16(), B.bfloat16()
    scale = torch.from_numpy((2.0 ** (np.ceil(np.log2(S)) + 3)).astype(np.float32)).to(dev)[:, None].expand(n, o).contiguous()
    zero, W0 = torch.zeros(o, device=dev), torch.zeros((o, i), device=dev, dtype=torch.bfloat16)
    errors, ws = torch.zeros((n, 4), device=dev), torch.zeros(256, dtype=torch.uint8, device=dev)
    for q in range(n):
        binding.l4q_quant_errors(desc, W0, A[q], B[q], scale[q], zero, errors[q], ws)
    torch.cuda.synchronize()
    off = np.abs(errors[:, 0].cpu().numpy().astype(np.float64) - np.abs(exact)) / (U * S)
    print(f"rank {r} {kind}: at most {off.max():.2f} u S", flush=True)
    # the share of D = 4 r u S that the kernel leaves to the matrix ops: 2 u S of every product, 2 u S of every step of 4, and
    # again of the two steps of zeros that end a rank of 8 mod 16
    assert off.max() <= 2 * r + 2 * (r // 4 + (2 if r % 16 else 0))


# ---- codes.  Weights on rounding ties, moved off them by a rank sum whose large products cancel exactly: the stated sum's own
# rounding errors decide the code.
CASES = [(96, 40, 8, 32, 4, 2.0, -6), (320, 72, 16, 64, 3, 1.5, -6), (128, 72, 24, 64, 4, 2.0, -6), (256, 136, 64, 128, 2, 2.0, -6),
         (256, 64, 72, 256, 4, 0.75, -6), (128, 40, 16, 64, 4, 2.0, -20)]  # (the last: subnormal factors)


def cancelling(i, o, r, g, bits, gamma, s_exp, ties):
    spec = LayerSpec(f"cancel{ties}_{o}x{i}_r{r}_b{bits}", 8, i, o, r, gamma * r, bits, g, DTYPE_BF16)
    rng = np.random.default_rng(i + r + bits)
    arrs = inputs.make_layer_inputs(spec, seed=r)
    step = 2.0 ** s_exp
    h = (r - 2) // 2
    A, B = np.zeros((r, i)), np.zeros((o, r))
    A[1:1 + h] = rng.uniform(1, 8, (h, i)) * rng.choice([1.0, -1.0], (h, i))
    B[:, 1:1 + h] = rng.integers(16, 128, (o, h)) / 16.0 * rng.choice([1.0, -1.0], (o, h))
    perm = rng.permutation(h)
    A[1 + h:1 + 2 * h], B[:, 1 + h:1 + 2 * h] = A[1:1 + h][perm], -B[:, 1:1 + h][:, perm]
    sums = 2.0 ** round(np.log2(4096 / (gamma * 2 * h * 20)))  # gamma S about 2^12 steps
    A[1:] *= sums * step
    A[0], B[:, 0] = step * 2.0 ** -14 / gamma, rng.choice([1.0, -1.0], o)  # the exact sum: 2^-14 of a step to either side
    if s_exp < -10:  # B becomes subnormal, exactly: multiples of 2^-133
        A, B = A * 2.0 ** 129, B * 2.0 ** -129
    qp = 2 ** (bits - 1) - 1
    k = rng.integers(-qp, qp + 1, (o, i)).astype(np.float64)
    tie = np.zeros((o, i), bool)
    if ties < 0:
        tie[:] = True
    else:
        at = rng.permutation(min(o, 32) * min(i, 64))[:ties]
        tie[at // min(i, 64), at % min(i, 64)] = True
    arrs["W0"] = inputs.round_to_bf16(((k - 0.5 * tie) * step).astype(np.float32))
    arrs["A"], arrs["B"] = (inputs.round_to_bf16(v.astype(np.float32)) for v in (A, B))
    s, b = np.full((o, i // g), step, np.float32), np.zeros((o, i // g), np.float32)
    return spec, arrs, s, b


@pytest.mark.parametrize("i,o,r,g,bits,gamma,s_exp", CASES)
def test_cancelling_sums_need_the_bound(i, o, r, g, bits, gamma, s_exp):
    """A code taken from the exact sum, and nothing but roundings of the quotient allowed for, is another one than the stated."""
    spec, arrs, s, b = cancelling(i, o, r, g, bits, gamma, s_exp, -1)
    dec, _, _ = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    exact = np.asarray(arrs["W0"], np.float64) + gamma * (np.asarray(arrs["B"], np.float64) @ np.asarray(arrs["A"], np.float64))
    w = np.clip(exact / 2.0 ** s_exp, -2.0 ** (bits - 1), 2.0 ** (bits - 1) - 1)
    code = np.rint(w)
    settled = np.abs(w - code) < 0.5 - 8 * U * (2 ** (bits - 1) + 1)
    assert ((code != dec.codes) & settled).sum() > 0.01 * o * i


@pytest.mark.gpu
@pytest.mark.parametrize("ties", [1, 5, 40, -1])
@pytest.mark.parametrize("i,o,r,g,bits,gamma,s_exp", CASES)
def test_cancelling_sums(i, o, r, g, bits, gamma, s_exp, ties):
    import torch
    from paper_2402_04902_amd import binding
    from parity_util import check_workspace_state
    from test_gpu_quantized_path import packed_on_gpu
    spec, arrs, s, b = cancelling(i, o, r, g, bits, gamma, s_exp, ties)
    print("case", spec.name, flush=True)
    layer = binding.upload(spec, arrs, s, b)
    dec, _, w32 = O.decide_f32(arrs["W0"], arrs["A"], arrs["B"], s, b, bits, g, spec.alpha)
    layer.forward()
    layer.backward()
    torch.cuda.synchronize()
    check_workspace_state(spec, layer, dec, w32, s, b, fused=r <= 32)
    got = packed_on_gpu(spec, layer).cpu().numpy().view(np.uint32)
    assert np.array_equal(got, O.pack_codes(dec.codes, bits))
