"""What a trace says of the row-wise kernels: launches that happened, and the bytes that they move."""
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch,group,recompute,res32", [("gpt", 3, 0, 0), ("llama", 3, 0, 1), ("llama", 1, 1, 1), ("bert", 1, 0, 1)])
def test_traced_launches_and_bytes(arch, group, recompute, res32):
    L, h, n_mb = 2, 256, 3
    cfg = P.StageConfig.make(arch=arch, n_layers=L, hidden=h, n_heads=4, head_dim=64, ffn=512, seq=128, mb=1, n_mb=n_mb, max_in_flight=group,
                             wgrad_group=group, recompute=recompute, residual_fp32=res32)
    st = P.Stage(cfg)
    st.zero_grads()
    st.trace_begin()
    for m in range(n_mb):
        x, dy = (torch.randn(128, h, device="cuda").bfloat16() for _ in range(2))
        st.forward(m % group, x, torch.empty_like(x))
        st.backward(m % group, dy, torch.empty_like(dy))
    st.flush_grads()
    sites = {s["name"]: s for s in st.trace_end()}
    # column sums of dqkv once per layer and micro-batch (where there are biases), one folding launch per layer and group
    folds = L * n_mb // group
    assert sites["colsum"]["launches"] == folds + (0 if arch == "llama" else L * n_mb)
    T, stream = 128, 4 if res32 else 2
    fwd, bwd = sites["norm_fwd"], sites["norm_bwd"]
    assert fwd["launches"] == 2 * L * n_mb * (2 if recompute else 1) and bwd["launches"] == 2 * L * n_mb
    # the stage's input and, for a group, its output gradient are kept once per micro-batch: 2 bytes more than the norm by itself
    # (an fp32 stream's first norm reads bf16 and writes the fp32 copy)
    assert fwd["bytes_per_launch"] == pytest.approx((stream + 2) * T * h + 8 * T + 2 * T * h * n_mb / fwd["launches"])
    assert bwd["bytes_per_launch"] == pytest.approx((stream + 6) * T * h + 8 * T + (2 * T * h * n_mb / bwd["launches"] if group > 1 else 0))
    st.close()
