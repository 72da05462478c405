"""float32 path: the rows that a chunk of keys or query rows reads beyond its last one carry no weight, also where that
row holds infinities."""
import pytest
import torch

from oracle import sp_attn_oracle as orc
from paper_2511_18871_amd import binding as B
from parity import to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [2, 33, 45, 64, 65, 97, 131])
def test_an_infinite_last_row_stays_infinite(T, d):
    gen = torch.Generator().manual_seed(T)
    q, k, v, d_o = (torch.randn(T, 2, d, generator=gen) for _ in range(4))
    v[T - 1] = float("inf")                              # seen by the last row alone
    d_o[T - 1] = float("inf")                            # reaches the dv of every key
    args = (1, [T - 1], d ** -0.5)
    o, lse = B.sp_attn_fwd(q.cuda(), k.cuda(), v.cuda(), *args)
    torch.cuda.synchronize()
    assert torch.all(o[T - 1] == float("inf"))
    finite = v.clone()
    finite[T - 1] = 0
    ro, _ = orc.sp_attn_fwd(to64(q), to64(k), to64(finite), *args)
    assert float(abs(to64(o)[:T - 1] - ro[:T - 1]).max()) <= 1e-5
    _, _, dv = B.sp_attn_bwd(q.cuda(), k.cuda(), finite.cuda(), o.nan_to_num(0, 0, 0), lse, d_o.cuda(), *args)
    torch.cuda.synchronize()
    assert torch.all(dv == float("inf"))
