"""GeLU and its derivative where u^3 no longer fits fp32 (u from 1e13 on): u and 0, 1 and 0, as for any other large u."""
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu

BIG = [1e4, 1e9, 1.2e13, 4e14, 1e16, 1e18]


@pytest.mark.parametrize("hidden,ffn,mb", [(256, 256, 1), (256, 4224, 4)])     # a tile whose waves share k, and one with the rolled epilogue
def test_gelu_of_large_preactivations(hidden, ffn, mb):
    """A bias of +-B in some columns makes u = +-B there to bf16 precision; the second matrix's row is scaled by 1 / B.  du of such a
    column is dy . w2, rounded to bf16, and its column sum the bias gradient: the terms' roundings are independent, 2^-9 / sqrt(3) =
    1.1e-3 of their norm together; 5e-3."""
    T = mb * 128
    cfg = P.StageConfig.make(arch="gpt", n_layers=1, hidden=hidden, n_heads=2, head_dim=64, ffn=ffn, seq=128, mb=mb)
    st = P.Stage(cfg)
    g = torch.Generator(device="cuda").manual_seed(3)
    st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.05)
    b1, w2 = st.param_view(0, "b1"), st.param_view(0, "w2")
    cols = []
    for i, B in enumerate(BIG):
        for sign in (1, -1):
            c = 5 + 17 * i + (8 if sign < 0 else 0)
            b1[c] = sign * B
            w2[c] = (w2[c].float() / B).bfloat16()
            cols.append((c, sign, B))
    x, dy = (torch.randn(T, hidden, generator=g, device="cuda").bfloat16() for _ in range(2))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    st.forward(0, x, y)
    st.backward(0, dy, dx)
    st.flush_grads()
    torch.cuda.synchronize()
    gb1 = st.grad_view(0, "b1")
    assert torch.isfinite(y).all() and torch.isfinite(dx).all() and torch.isfinite(st.grads).all()
    for c, sign, B in cols:
        if sign < 0:
            assert gb1[c] == 0, (c, B)
            continue
        du = dy.double() @ w2[c].double()
        assert abs(gb1[c].double() - du.sum()) <= 5e-3 * du.norm(), (c, B)
    st.close()
