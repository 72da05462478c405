"""Rows of the log-probability passes at every cut a row can have: elements ahead of a 16-byte boundary (odd vocabularies), vectors around whole rounds
of each workgroup size, a tail; prompt rows of a gradient that the call allocates are zero."""
import numpy as np
import pytest
import torch

from oracle import loss_oracle as lo
from paper_2511_18871_amd import binding as B

pytestmark = pytest.mark.gpu

PACK = ([3, 0, 2], [2, 1, 2], [1, 3, 2, 4, 1])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [1, 7, 8, 9, 1023, 2048, 4095, 4097, 8192, 16384, 16389, 49157])
def test_rows_of_any_vocabulary(V, dtype):
    pl, Gs, rl = PACK
    T = sum(pl) + sum(rl)
    gen = torch.Generator().manual_seed(V)
    z = (3.0 * torch.randn(T, V, generator=gen)).to(dtype)
    if V > 8:
        z[4, :V // 2] = float("-inf")                    # half a vocabulary masked
    y = torch.randint(V // 2, V, (T,), generator=gen, dtype=torch.int32)
    g = torch.randn(T, generator=gen)
    idx = lo.response_index(pl, Gs, rl)
    resp = idx >= 0
    z64 = z.to(torch.float64).numpy()
    rlogp, _ = lo.logprob_fwd(z64, y.numpy(), idx)
    rdz = lo.logprob_bwd(z64, y.numpy(), g.numpy().astype(np.float64), idx)
    logp, lse = B.sp_attn_logprob_fwd(z.cuda(), y.cuda(), pl, Gs, rl)
    dz = B.sp_attn_logprob_bwd(z.cuda(), y.cuda(), lse, g.cuda(), pl, Gs, rl)
    torch.cuda.synchronize()
    logp, dz = logp.cpu().double().numpy(), dz.cpu().double().numpy()
    assert np.all(logp[~resp] == 0.0) and np.all(dz[~resp] == 0.0)
    # fp32 accumulation over V terms, as in the tests of whole packings
    assert float(np.abs(logp[resp] - rlogp[resp]).max()) <= 2e-5
    err = np.abs(dz[resp] - rdz[resp])
    tol = 1e-5 * max(1.0, float(np.abs(rdz).max())) if dtype == torch.float32 else 2.0 ** -8 * np.abs(rdz[resp]) + 1e-5
    assert float((err - tol).max()) <= 0.0
