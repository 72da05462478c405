"""Rows of the log-probability passes at every cut a row can have: elements ahead of a 16-byte boundary (odd vocabularies),
vectors around whole rounds of each workgroup size (64 threads below 4096 bf16 or 2048 float32 elements, 1024 from 65536 or
32768 on, 256 between), a tail; masked rows; a gradient too large for the caches, which is stored past them; prompt rows of
a gradient that the call allocates are zero."""
import numpy as np
import pytest
import torch

from oracle import loss_oracle as lo
from paper_2511_18871_amd import binding as B

pytestmark = pytest.mark.gpu

PACK = ([3, 0, 2], [2, 1, 2], [1, 3, 2, 4, 1])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [1, 7, 8, 9, 1023, 2048, 4095, 4097, 8192, 16384, 16389, 49157, 65535, 65536, 65543, 151936])
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


LOWEST = {torch.bfloat16: float(torch.finfo(torch.bfloat16).min), torch.float32: float(torch.finfo(torch.float32).min)}


@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 300), (torch.bfloat16, 4097), (torch.bfloat16, 65543),
                                     (torch.float32, 300), (torch.float32, 4097), (torch.float32, 40001)])
@pytest.mark.parametrize("mask", [-1e9, -1e10, -1e11, -1e12, -1e20, -1e30, -1e37, "lowest", float("-inf")])
def test_rows_masked_with_any_low_value(mask, dtype, V):
    """Rows of which a first part, a last part, all but one element or every element holds a mask value, and rows whose
    maximum is as large; one vocabulary per workgroup size."""
    mask = LOWEST[dtype] if mask == "lowest" else mask
    pl, Gs, rl = PACK
    T = sum(pl) + sum(rl)
    gen = torch.Generator().manual_seed(V)
    z = (3.0 * torch.randn(T, V, generator=gen)).to(dtype)
    idx = lo.response_index(pl, Gs, rl)
    rows = np.flatnonzero(idx >= 0)
    y = torch.full((T,), V // 2, dtype=torch.int32)
    z[rows[0], :V // 2] = mask
    z[rows[1], V // 2 + 1:] = mask
    z[rows[2], :] = mask
    z[rows[2], V // 2] = 1.5
    whole = [rows[3], rows[4]]
    if np.isfinite(mask):
        z[rows[3], :] = mask                             # the whole row
        z[rows[4], :] = -mask                            # as large, positive
        z[rows[4], ::2] = mask
        z[rows[4], V // 2] = -mask
    z[rows[5], 1::2] = mask
    z[rows[5], V // 2] = 0.25
    g = torch.randn(T, generator=gen)
    z64 = z.to(torch.float64).numpy()
    rlogp, rlse = lo.logprob_fwd(z64, y.numpy(), idx)
    rdz = lo.logprob_bwd(z64, y.numpy(), g.numpy().astype(np.float64), idx)
    logp, lse = B.sp_attn_logprob_fwd(z.cuda(), y.cuda(), pl, Gs, rl)
    dz = B.sp_attn_logprob_bwd(z.cuda(), y.cuda(), lse, g.cuda(), pl, Gs, rl)
    torch.cuda.synchronize()
    logp, lse, dz = logp.cpu().double().numpy(), lse.cpu().double().numpy(), dz.cpu().double().numpy()
    assert np.all(np.isfinite(lse[rows])) and np.all(np.isfinite(logp[rows])) and np.all(np.isfinite(dz[rows]))
    # fp32: the sum as in the tests above; where the row's maximum is large, lse itself (and logp, a difference from it) is
    # rounded to a spacing of float32
    tol = 2e-5 + 2.0 ** -23 * np.abs(rlse[rows])
    assert np.all(np.abs(lse[rows] - rlse[rows]) <= tol)
    assert np.all(np.abs(logp[rows] - rlogp[rows]) <= tol)
    keep = [t for t in rows if t not in whole]           # exp(z - lse) has no digits where lse is rounded that coarsely
    err = np.abs(dz[keep] - rdz[keep])
    gtol = 1e-5 * max(1.0, float(np.abs(rdz).max())) if dtype == torch.float32 else 2.0 ** -8 * np.abs(rdz[keep]) + 1e-5
    assert float((err - gtol).max()) <= 0.0


@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 151936), (torch.bfloat16, 151937), (torch.bfloat16, 20001), (torch.float32, 75968),
                                     (torch.float32, 75971), (torch.float32, 1501)])
def test_a_gradient_beyond_the_caches(dtype, V):
    size = 2 if dtype == torch.bfloat16 else 4
    n = (256 << 20) // (V * size) // 4 + 1               # tokens: 4 n + 14, just over 256 MB
    pl, Gs, rl = [n, 3], [2, 1], [n, n + 9, n + 2]
    T = sum(pl) + sum(rl)
    assert T * V * size > 256 << 20
    gen = torch.Generator(device="cuda").manual_seed(V)
    z = torch.empty(T, V, dtype=dtype, device="cuda").normal_(0.0, 3.0, generator=gen)
    y = torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32)
    g = torch.randn(T, generator=gen, device="cuda")
    stale = torch.full_like(z, float("nan"))             # what the call's own allocation may hold
    del stale
    logp, lse = B.sp_attn_logprob_fwd(z, y, pl, Gs, rl)
    dz = B.sp_attn_logprob_bwd(z, y, lse, g, pl, Gs, rl)
    torch.cuda.synchronize()
    idx = lo.response_index(pl, Gs, rl)
    assert not dz[torch.from_numpy(idx < 0).cuda()].any()
    assert torch.isfinite(dz).all()
    at = np.flatnonzero(idx >= 0)
    rows = at[np.linspace(0, len(at) - 1, 12).astype(int)]
    pick = lambda x: x[torch.from_numpy(rows).cuda()].cpu().double().numpy()
    z64 = pick(z)
    rlogp, _ = lo.logprob_fwd(z64, y.cpu().numpy()[rows], idx[rows])
    rdz = lo.logprob_bwd(z64, y.cpu().numpy()[rows], pick(g), idx[rows])
    assert float(np.abs(pick(logp) - rlogp).max()) <= 2e-5
    err = np.abs(pick(dz) - rdz)
    tol = 1e-5 * max(1.0, float(np.abs(rdz).max())) if dtype == torch.float32 else 2.0 ** -8 * np.abs(rdz) + 1e-5
    assert float((err - tol).max()) <= 0.0
