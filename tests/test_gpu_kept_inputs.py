"""The copies of a stage's input and output gradient that the norm kernels leave behind."""
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch", ["gpt", "llama"])
@pytest.mark.parametrize("res32", [0, 1])
@pytest.mark.parametrize("hidden,seq", [(256, 128), (640, 384), (1024, 256), (2048, 128), (4096, 256), (5120, 128), (8192, 128),
                                        (8320, 128), (16384, 128)])
def test_input_is_kept(arch, res32, hidden, seq):
    """Every number of chunks per lane, and a block per row (over 8192 columns): the slot holds the input bit for bit, also where
    the caller's buffer is overwritten by the output."""
    cfg = P.StageConfig.make(arch=arch, n_layers=1, hidden=hidden, n_heads=2, head_dim=64, ffn=128, seq=seq, mb=3, max_in_flight=2, residual_fp32=res32)
    st = P.Stage(cfg)
    g = torch.Generator(device="cuda").manual_seed(1)
    st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.05)
    xs = [torch.randn(3 * seq, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    ys = []
    for slot, x in enumerate(xs):
        y = torch.empty_like(x)
        st.forward(slot, x, y)
        assert torch.equal(st.layer_input(slot, 0).to(torch.bfloat16), x)
        ys.append(y)
    st.backward(0, torch.zeros_like(xs[0]), torch.empty_like(xs[0]))
    in_place = xs[0].clone()
    st.forward(0, in_place, in_place)
    assert torch.equal(in_place, ys[0]) and torch.equal(st.layer_input(0, 0).to(torch.bfloat16), xs[0])
    st.close()


@pytest.mark.parametrize("arch", ["gpt", "llama"])
@pytest.mark.parametrize("hidden,heads", [(256, 4), (640, 10), (1024, 16), (4096, 2), (4224, 2), (8320, 2)])
@pytest.mark.parametrize("defer", ["0", "1"])
def test_output_gradient_is_kept(arch, hidden, heads, defer, monkeypatch):
    """Groups of two, the caller's gradient overwritten by dx and again before its group is closed: the weight gradients are
    those of gradients left alone, bit for bit."""
    monkeypatch.setenv("AH_DEFER_WGRADS", defer)             # both read when the stage is created; "0" takes the second stream
    monkeypatch.setenv("AH_SIDE_STREAM_MIN_GFLOP", "0")
    res = []
    for in_place in (False, True):
        cfg = P.StageConfig.make(arch=arch, n_layers=2 if hidden < 2048 else 1, hidden=hidden, n_heads=heads, head_dim=64, ffn=256, seq=128,
                                 mb=3, n_mb=3, max_in_flight=2, wgrad_group=2)
        st = P.Stage(cfg)
        g = torch.Generator(device="cuda").manual_seed(2)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.05)
        st.zero_grads()
        dxs = []
        for m in range(3):
            x, dy = (torch.randn(384, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
            dx = dy if in_place else torch.empty_like(dy)
            st.forward(m % 2, x, torch.empty_like(x))
            st.backward(m % 2, dy, dx)
            dxs.append(dx.clone())
            if in_place:
                dy.fill_(float("nan"))
        st.flush_grads()
        res.append(dxs + [st.grads.clone()])
        st.close()
    assert torch.isfinite(res[0][-1]).all()
    assert all(torch.equal(a, b) for a, b in zip(*res))
