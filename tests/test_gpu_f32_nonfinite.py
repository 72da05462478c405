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


# a NaN among the keys reaches every row that sees it, also where it is alone in a chunk of keys, and no other row
@pytest.mark.parametrize("d,heads", [(64, 2), (64, 56), (128, 2), (128, 12)])         # eight waves per row, blocks of 16 rows
@pytest.mark.parametrize("key", [0, 31, 63, 64, 65, 104])
def test_a_nan_key_reaches_the_rows_that_see_it(key, d, heads):
    prompt, resp = 64, [1, 40]
    T, gen = prompt + sum(resp), torch.Generator().manual_seed(key)
    q, k, v = (torch.randn(T, heads, d, generator=gen) for _ in range(3))
    args = (prompt, resp, d ** -0.5)
    clean, _ = B.sp_attn_fwd(q.cuda(), k.cuda(), v.cuda(), *args)
    k[key] = float("nan")
    o, lse = B.sp_attn_fwd(q.cuda(), k.cuda(), v.cuda(), *args)
    torch.cuda.synchronize()
    t = torch.arange(T)
    start = torch.where(t < prompt, 0, torch.where(t < prompt + resp[0], prompt, prompt + resp[0]))
    sees = ((key <= t) & ((key < prompt) | (key >= start))).cuda()
    assert o[sees].isnan().all() and lse[:, sees].isnan().all()
    assert torch.equal(o[~sees], clean[~sees]) and lse[:, ~sees].isfinite().all()


@pytest.mark.parametrize("d,heads", [(64, 2), (64, 56), (128, 2), (128, 12)])
def test_a_chunk_of_nan_keys_is_not_passed_over(d, heads):
    T, gen = 200, torch.Generator().manual_seed(d)
    q, k, v = (torch.randn(T, heads, d, generator=gen) for _ in range(3))
    k[:64] = float("nan")
    o, lse = B.sp_attn_fwd(q.cuda(), k.cuda(), v.cuda(), T, [], d ** -0.5)
    torch.cuda.synchronize()
    assert o.isnan().all() and lse.isnan().all()


@pytest.mark.parametrize("d", [64, 128])
def test_a_nan_key_of_a_short_group_stays_in_its_group(d):
    """Rows by a wave each (a block of 16 would span two groups)."""
    n, prompt, resp, heads = 24, 7, [3, 1], 8
    T, pack, gen = n * 11, ([prompt] * n, [2] * n, resp * n), torch.Generator().manual_seed(d)
    assert B.sp_attn_f32_rows(*pack, heads, heads, d)[0] == 4
    q, k, v = (torch.randn(T, heads, d, generator=gen) for _ in range(3))
    clean, _ = B.sp_attn_fwd_batched(q.cuda(), k.cuda(), v.cuda(), *pack, d ** -0.5)
    key = 5 * 11 + 8                                     # the second token of the sixth group's first response
    k[key] = float("nan")
    o, lse = B.sp_attn_fwd_batched(q.cuda(), k.cuda(), v.cuda(), *pack, d ** -0.5)
    torch.cuda.synchronize()
    sees = torch.zeros(T, dtype=torch.bool, device="cuda")
    sees[key:key + 2] = True
    assert o[sees].isnan().all() and lse[:, sees].isnan().all()
    assert torch.equal(o[~sees], clean[~sees]) and lse[:, ~sees].isfinite().all()
