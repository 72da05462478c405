"""Calls that read the segment table from their kernel's arguments (up to 768 words) or from the workspace, and the objective of
up to 16 responses in one launch or of more in two."""
import numpy as np
import pytest
import torch

from oracle import loss_oracle as lo
from oracle import rope_oracle as rope
from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import to64

pytestmark = pytest.mark.gpu


def packing(words, n_groups):
    """Lengths whose table has `words` words: 4, 8 per group, one per response and group."""
    n_resp = words - 4 - 9 * n_groups
    Gs = [n_resp // n_groups + (g < n_resp % n_groups) for g in range(n_groups)]
    rng = np.random.default_rng(words)
    return [int(rng.integers(1, 9)) for _ in Gs], Gs, [int(rng.integers(0, 5)) for _ in range(n_resp)]


@pytest.mark.parametrize("words", [13, 767, 768, 769])
def test_rope_and_loss_around_the_argument_limit(words):
    pl, Gs, rl = packing(words, 1 if words == 13 else 40)
    assert len(B.sp_attn_segment_table(pl, Gs, rl)) == words
    T = sum(pl) + sum(rl)
    gen = torch.Generator().manual_seed(words)
    x = torch.randn(T, 2, 64, generator=gen)
    want = rope.rope_rotate(to64(x), rope.positions_batched(pl, Gs, rl), 1e4)
    got = to64(B.sp_attn_rope(x.cuda(), pl, Gs, rl, 1e4))
    assert float(np.abs(got - want).max()) <= 2e-6 * max(1.0, float(np.abs(want).max()))
    idx = lo.response_index(pl, Gs, rl)
    z, y = 2.0 * torch.randn(T, 96, generator=gen), torch.randint(0, 96, (T,), generator=gen, dtype=torch.int32)
    logp, lse = B.sp_attn_logprob_fwd(z.cuda(), y.cuda(), pl, Gs, rl)
    g = torch.randn(T, generator=gen)
    dz = B.sp_attn_logprob_bwd(z.cuda(), y.cuda(), lse, g.cuda(), pl, Gs, rl)
    torch.cuda.synchronize()
    resp = idx >= 0
    rlogp, _ = lo.logprob_fwd(z.double().numpy(), y.numpy(), idx)
    assert not resp.any() or float(np.abs(logp.cpu().double().numpy() - rlogp)[resp].max()) <= 2e-5
    rdz = lo.logprob_bwd(z.double().numpy(), y.numpy(), g.double().numpy(), idx)
    assert float(np.abs(dz.cpu().double().numpy() - rdz).max()) <= 2e-5 * max(1.0, float(np.abs(rdz).max()))


@pytest.mark.parametrize("n_resp", [0, 1, 15, 16, 17, 300])
def test_grpo_one_launch_and_two(n_resp):
    rng = np.random.default_rng(n_resp)
    pl, Gs, rl = [5, 3], [n_resp // 2, n_resp - n_resp // 2], [int(rng.integers(0, 90)) for _ in range(n_resp)]
    T = sum(pl) + sum(rl)
    gen = torch.Generator().manual_seed(n_resp)
    logp = -torch.rand(T, generator=gen) * 3 - 0.05
    old, ref = logp + 0.4 * torch.randn(T, generator=gen), logp + 0.3 * torch.randn(T, generator=gen)
    adv = torch.randn(max(1, n_resp), generator=gen)[:n_resp]
    idx = lo.response_index(pl, Gs, rl)
    loss, g = B.sp_attn_grpo_loss(logp.cuda(), old.cuda(), ref.cuda(), adv.cuda() if n_resp else torch.zeros(1).cuda(), pl, Gs, rl,
                                  0.2, 0.2, 0.02)
    torch.cuda.synchronize()
    if n_resp == 0:
        assert loss.item() == 0.0
        return
    rloss, rg = lo.grpo_loss(logp.numpy(), old.numpy(), ref.numpy(), adv.numpy(), idx, 0.2, 0.2, 0.02)
    resp = idx >= 0
    assert abs(loss.item() - rloss) <= 1e-5 * max(1.0, abs(rloss))
    assert not resp.any() or float(np.abs(g.cpu().double().numpy() - rg)[resp].max()) <= 1e-5 * max(1.0, float(np.abs(rg).max()))
