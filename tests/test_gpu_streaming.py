"""Rotations and logit gradients at the edges of a workgroup's heads and tokens, and at the sizes from which they read or store
past the caches."""
import numpy as np
import pytest
import torch

from oracle import rope_oracle as rope
from paper_2511_18871_amd import binding as B
from parity import to64

pytestmark = pytest.mark.gpu
PACK = ([37, 0, 1], [2, 3, 0], [5, 64, 1, 0, 130])       # 238 tokens


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(1, 1), (7, 1), (8, 8), (9, 1), (40, 8), (41, 7), (48, 1), (100, 4)])
def test_rope_heads(d, hq, hkv):
    gen = torch.Generator().manual_seed(hq)
    q, k = torch.randn(238, hq, d, generator=gen), torch.randn(238, hkv, d, generator=gen)
    pos = rope.positions_batched(*PACK)
    got = B.sp_attn_rope_qk(q.cuda(), k.cuda(), *PACK, 1e4)
    for x, y in zip((q, k), got):
        ref = rope.rope_rotate(to64(x), pos, 1e4)
        assert float(np.abs(to64(y) - ref).max()) <= 2e-6 * max(1.0, float(np.abs(ref).max()))


def test_rope_of_a_large_tensor_equals_its_parts():
    # 252 MB and 63 MB of outputs
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(24601, 40, 128, generator=gen, device="cuda").to(torch.bfloat16)
    pack = ([20001], [2], [4000, 600], 1e6)
    y = B.sp_attn_rope(x, *pack)
    for h in range(0, 40, 10):
        part = B.sp_attn_rope(x[:, h:h + 10].contiguous(), *pack)
        assert torch.equal(y[:, h:h + 10], part)


@pytest.mark.parametrize("T,V", [(900, 50001), (3000, 50000), (3000, 50001), (140000, 1003)])       # 90 MB; 300 MB and 281 MB: past the caches
@pytest.mark.parametrize("dtype", [torch.bfloat16])
def test_logit_gradients_of_large_logits(T, V, dtype):
    gen = torch.Generator(device="cuda").manual_seed(V)
    z = torch.randn(T, V, generator=gen, device="cuda").to(dtype)
    y = torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32)
    g = torch.randn(T, generator=gen, device="cuda")
    pack = ([100], [2], [T - 200, 100])
    _, lse = B.sp_attn_logprob_fwd(z, y, *pack)
    dz = B.sp_attn_logprob_bwd(z, y, lse, g, *pack)
    assert not dz[:100].any()
    for a in range(100, T, 500):
        zz = z[a:a + 500].double()
        ref = -torch.softmax(zz, 1)
        ref[torch.arange(len(zz)), y[a:a + 500].long()] += 1
        ref *= g[a:a + 500, None].double()
        # bf16 rounding of the result (2^-8 of it), and float32 exponentials of differences near -lse (1e-6 of it)
        assert bool(((dz[a:a + 500].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-6 * g[a:a + 500, None].abs().double()).all())
