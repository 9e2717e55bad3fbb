"""Attention under the mask: what is not finite in a later position leaves earlier rows as they are, bit for bit.

A probability of exactly zero times an infinite value is a NaN, so a block of positions that lies wholly behind the mask must be
skipped, not multiplied by zero.  The kernels skip by 64 positions (launches of more than 256 blocks of 128 rows) or by 32."""
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,S,nh,block", [(2, 128, 3, 32), (1, 512, 2, 32), (2, 128, 130, 64), (1, 384, 88, 64)])
def test_rows_before_a_bad_position_are_untouched(B, S, nh, block, d, bad):
    T, hl = B * S, nh * d
    g = torch.Generator().manual_seed(S + d)
    qkv, d_o = (torch.randn(T, n, generator=g).bfloat16().cuda() for n in (3 * hl, hl))

    def call(qkv, d_o, stats=None):
        o = torch.empty(T, hl, dtype=torch.bfloat16, device="cuda")
        dqkv = torch.empty(T, 3 * hl, dtype=torch.bfloat16, device="cuda")
        lse, delta = (torch.empty(B, nh, S, device="cuda") for _ in range(2))
        P.attention_fwd(qkv, o, lse, B, S, nh, d, True)
        fwd = (o, lse)
        P.attention_bwd(qkv, *(stats or fwd), d_o, dqkv, delta, B, S, nh, d, True)
        return fwd, dqkv.view(B, S, 3, nh * d), delta

    clean, grads, delta = call(qkv, d_o)
    assert all(torch.isfinite(t).all() for t in (*clean, grads))
    for p in sorted({40, 64, 127, S // 2 + 33, S - 1}):
        first, after = p // block * block, (p // block + 1) * block      # the block of p
        # keys and values of position p: queries of earlier blocks see neither
        x = qkv.clone().view(B, S, 3, hl)
        x[:, p, 1:] = bad
        (o, lse), dq, dlt = call(x.view(T, 3 * hl), d_o, clean)
        assert torch.equal(o.view(B, S, hl)[:, :first], clean[0].view(B, S, hl)[:, :first]), p
        assert torch.equal(lse[:, :, :first], clean[1][:, :, :first]), p
        assert torch.equal(dq[:, :first, 0], grads[:, :first, 0]), p
        assert torch.equal(dlt, delta), p
        # query and output gradient of position p: keys of later blocks are not seen by it
        x, y = qkv.clone().view(B, S, 3, hl), d_o.clone().view(B, S, hl)
        x[:, p, 0] = bad
        y[:, p] = bad
        _, dkv, _ = call(x.view(T, 3 * hl), y.view(T, hl), clean)
        assert torch.equal(dkv[:, after:, 1:], grads[:, after:, 1:]), p
