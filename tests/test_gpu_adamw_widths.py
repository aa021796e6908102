"""The AdamW step at sizes on both sides of its rule: four elements per thread where every tensor's size is a
multiple of 4, one element per thread otherwise."""
import numpy as np
import pytest

from paper_2402_04902_amd import binding
from paper_2402_04902_amd.inputs import DTYPE_BF16, DTYPE_F32, LayerSpec

# (in, out, rank, group, type): the tensors hold rank x in, out x rank and twice out x in / group elements.
SHAPES = [(64, 4, 1, 64, DTYPE_F32),       # the smallest sizes of the wide form: 64, 4, 4, 4
          (64, 137, 1, 64, DTYPE_F32),     # 64, 137, 137, 137: one element per thread
          (128, 6, 2, 64, DTYPE_F32),      # 128, 12, 12, 12: tensors end inside a wave of the wide form
          (192, 130, 3, 64, DTYPE_F32),    # 576, 390, 390, 390: only the first a multiple of 4
          (64, 8, 1, 64, DTYPE_BF16),      # 64, 8, 8, 8
          (1024, 520, 5, 64, DTYPE_BF16)]  # several workgroups, the last one partly filled


@pytest.mark.gpu
@pytest.mark.parametrize("n_in,n_out,rank,group,dtype", SHAPES)
def test_adamw_step_at_odd_and_even_sizes(n_in, n_out, rank, group, dtype):
    import torch
    from oracle import optim_oracle as OO
    spec = LayerSpec("adamw", 8, n_in, n_out, rank, 8.0, 4, group, dtype)
    rng = np.random.default_rng(n_out)
    shapes = [(rank, n_in), (n_out, rank), (n_out, spec.groups), (n_out, spec.groups)]
    dev = torch.device("cuda:0")
    params = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    grads = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    n = sum(p.size for p in params)
    m0 = rng.standard_normal(n).astype(np.float32) * 0.1
    v0 = rng.random(n).astype(np.float32)
    tp = [torch.from_numpy(p.copy()).to(dev) for p in params]
    tg = [torch.from_numpy(g).to(dev) for g in grads]
    # 8 more elements than the moments need: they must be left alone.
    m = torch.from_numpy(np.concatenate([m0, np.full(8, 3.0, np.float32)])).to(dev)
    v = torch.from_numpy(np.concatenate([v0, np.full(8, 5.0, np.float32)])).to(dev)
    copies = [torch.zeros(s, dtype=torch.bfloat16, device=dev) for s in shapes[:2]] if dtype == DTYPE_BF16 else [None] * 2
    binding.l4q_adamw_step(binding.make_desc(spec), binding.L4QAdamW(1e-3, 0.9, 0.999, 1e-8, 0.01, 3), *tp, *tg, m, v,
                           *copies)
    torch.cuda.synchronize()
    at = 0
    for k in range(4):
        size = params[k].size
        want = OO.adamw_step(params[k].astype(np.float64).ravel(), grads[k].ravel(), m0[at:at + size].astype(np.float64),
                             v0[at:at + size].astype(np.float64), 1e-3, 0.9, 0.999, 1e-8, 0.01, 3)
        got = [tp[k].cpu().numpy().ravel(), m[at:at + size].cpu().numpy(), v[at:at + size].cpu().numpy()]
        for a, b in zip(got, want):   # about ten fp32 operations, none of which cancels by more than a few digits
            assert np.allclose(a, b, rtol=2e-5, atol=1e-7), (k, np.abs(a - b).max())
        at += size
    assert torch.all(m[n:] == 3.0) and torch.all(v[n:] == 5.0)
    for k in range(2 if dtype == DTYPE_BF16 else 0):
        assert torch.equal(copies[k], tp[k].to(torch.bfloat16))
