"""The column sums behind the QKV bias gradient ride along with the first norm's backward in small stages on one stream, and are a launch of
their own in a trace: the same bits, for both norm kernels (rows up to 1024 wide, and wider), one micro-batch and a group's sums."""
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch,hidden,heads,seq,mb,group", [("gpt", 256, 2, 128, 1, 1), ("bert", 640, 5, 128, 3, 3), ("gpt", 1152, 10, 384, 1, 2),
                                                            ("gpt", 4224, 2, 128, 1, 1)])
def test_same_bits_as_a_launch_of_their_own(arch, hidden, heads, seq, mb, group):
    cfg = P.StageConfig.make(arch=arch, n_layers=2, hidden=hidden, n_heads=heads, head_dim=128, ffn=256, seq=seq, mb=mb, n_mb=3,
                             max_in_flight=group, wgrad_group=group)
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).bfloat16()
    st = P.Stage(cfg)
    assert st.backward_streams() == 1
    st.params.copy_(rnd(st.params.numel(), std=0.05))
    xs, dys = ([rnd(mb * seq, hidden) for _ in range(3)] for _ in range(2))
    got = []
    for traced in (True, False):
        st.grads.fill_(float("nan"))
        st.zero_grads()
        if traced:
            st.trace_begin()
        for m in range(3):
            st.forward(m % group, xs[m], torch.empty_like(xs[m]))
            st.backward(m % group, dys[m], torch.empty_like(xs[m]))
        st.flush_grads()
        if traced:
            st.trace_end()
        torch.cuda.synchronize()
        got.append(st.grads.clone())
    assert torch.isfinite(got[0]).all() and torch.equal(got[0], got[1])
    for l in range(2):
        assert float(st.grad_view(l, "bqkv").abs().max()) > 0
    st.close()
