"""The attention kernels' rings: a slot that is filled before every wave has read it shows as a result that changes from call to
call (a wave that lags behind the others by the time of a load reads later rows).  Every form, many blocks, compared bit for bit."""
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,nh", [(2, 128, 130), (2, 640, 26), (2, 2048, 16),      # 128-row kernels
                                    (1, 256, 16), (1, 2048, 16)])                  # 64-row kernels
def test_results_do_not_change_from_call_to_call(B, S, nh, d, causal):
    T, hl = B * S, nh * d
    g = torch.Generator().manual_seed(S)
    qkv, d_o = (torch.randn(T, n, generator=g).bfloat16().cuda() for n in (3 * hl, hl))
    first = None
    for call in range(40):
        o = torch.empty(T, hl, dtype=torch.bfloat16, device="cuda")
        dqkv = torch.empty(T, 3 * hl, dtype=torch.bfloat16, device="cuda")
        lse, delta = (torch.empty(B, nh, S, device="cuda") for _ in range(2))
        P.attention_fwd(qkv, o, lse, B, S, nh, d, causal)
        P.attention_bwd(qkv, o, lse, d_o, dqkv, delta, B, S, nh, d, causal)
        got = (o, lse, dqkv, delta)
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first)), call
