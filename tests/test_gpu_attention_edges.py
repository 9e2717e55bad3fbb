"""Attention at the sequence lengths where the kernels' pipelines begin and end: one query block (the first tile is already a masked
one), two, an odd number, a few rounds; over more than 256 blocks of 128 rows, and over fewer, which take the 64-row kernels.

Tolerances.  Output: probabilities and result are rounded to bf16 once each, 2^-9 / sqrt(3) = 1.1e-3 of a row's norm per
rounding; 4e-3.  Log-sum-exp: fp32 sums and the hardware's exponential, 1e-6 of values below 10; 1e-4.  Gradients, by blocks
of 32 rows (one wave's): P, dS and the result are rounded, 2e-3 together, and for dQ and dK delta_i comes from the rounded output, an
error of 2^-9 |do_i| |o_i| / sqrt(3) in each dS of the row: small beside a dS of many keys (3.3e-3 measured for every block;
1e-2 allowed), but for a query with two or three keys a sizeable part of the row (0.18 seen for one row), which is below 0.18 /
sqrt(32) = 0.03 of its block; 0.06 for the first block of the masked dQ and dK.  A wrong row has error 1, its block 1 / sqrt(32) = 0.18.

Rows leave through LDS in pieces of 8 elements, and one of them is lost in a block's norm: each against the block's root mean
square.  The largest of a block's few hundred pieces is within about six times the block's error (2.7e-2 measured); 0.1, and 0.5
where a row may be off by 0.18 (a row of few keys is up to twice its block's average).  A wrong piece has error 1.4."""
import numpy as np
import pytest
import torch

import paper_2512_20953_amd as P
from oracle import stage_ref as R
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _blocks(got, ref, rows=32):
    d, r = ((t.reshape(-1, rows * t.shape[-1]) ** 2).sum(1) for t in (got - ref, ref))
    return np.sqrt(d / np.maximum(r, U.FLOOR ** 2 * r.mean()))


def _pieces(got, ref, rows=32):
    """The worst piece of each block."""
    n = rows * ref.shape[-1]
    rms = np.sqrt((ref.reshape(-1, n) ** 2).mean(1))
    d = np.sqrt(((got - ref).reshape(-1, n // 8, 8) ** 2).mean(2)).max(1)
    return d / np.maximum(rms, U.FLOOR * np.sqrt((ref ** 2).mean()))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,nh", [(2, 128, 130), (3, 256, 44), (1, 384, 88), (2, 640, 26), (1, 1024, 34),      # 128-row kernels
                                    (1, 128, 2), (2, 256, 3), (1, 640, 5), (1, 1024, 4)])                       # 64-row kernels
def test_attention_edges(B, S, nh, d, causal):
    T, hl = B * S, nh * d
    g = torch.Generator().manual_seed(S + d)
    qkv, d_o = (torch.randn(T, n, generator=g).bfloat16().cuda() for n in (3 * hl, hl))
    o = torch.full((T, hl), float("nan"), dtype=torch.bfloat16, device="cuda")
    dqkv = torch.full((T, 3 * hl), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse, delta = (torch.full((B, nh, S), float("nan"), device="cuda") for _ in range(2))
    P.attention_fwd(qkv, o, lse, B, S, nh, d, causal)
    P.attention_bwd(qkv, o, lse, d_o, dqkv, delta, B, S, nh, d, causal)
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.isfinite(dqkv).all() and torch.isfinite(lse).all()
    for b, j in {(0, 0), (B - 1, nh - 1), (0, nh // 2)}:
        head = lambda t, blk=0: U.to_np(t[b * S:(b + 1) * S, blk * hl + j * d: blk * hl + (j + 1) * d])
        q, k, v = (head(qkv, blk) for blk in range(3))
        s = q @ k.T / np.sqrt(d)
        if causal:
            s[np.triu_indices(S, 1)] = -np.inf
        m = s.max(1)
        assert np.abs(lse[b, j].cpu().numpy() - (m + np.log(np.exp(s - m[:, None]).sum(1)))).max() <= 1e-4
        q, k, v, do = (t[None, None] for t in (q, k, v, head(d_o)))
        ref = R.attention_fwd(q, k, v, causal)[0, 0]
        assert _blocks(head(o), ref).max() <= 4e-3 and _pieces(head(o), ref).max() <= 0.1, (b, j)
        for blk, ref in enumerate(R.attention_bwd(q, k, v, do, causal)):
            eb, ep = (f(head(dqkv, blk), ref[0, 0]) for f in (_blocks, _pieces))
            if causal and blk < 2:
                assert eb[0] <= 0.06 and ep[0] <= 0.5, (b, j, blk)
                eb, ep = eb[1:], ep[1:]
            assert (eb <= 1e-2).all() and (ep <= 0.1).all(), (b, j, blk)
