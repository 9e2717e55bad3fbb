"""Tiles of 192 or 160 in an extent (forward and input gradient): each at the smallest product that takes it (asserted), then inside a
layer with the fused epilogues.  Where an epilogue writes pieces of a 96- or 80-wide strip, 48 or 40 of a wave's lanes hold one."""
import numpy as np
import pytest
import torch

import paper_2512_20953_amd as P
from synth import stage_inputs as SI
from tests import gpu_util as U
from tests.test_gpu_gemm_tiles import check_products

pytestmark = pytest.mark.gpu

SMALLEST = [(768, 6144, 128, (128, 192)), (1152, 4096, 256, (192, 128)), (1920, 5632, 384, (192, 256)), (3328, 2560, 2048, (256, 160)),
            (1536, 6144, 2048, (256, 192))]


def _tiles(layout, M, N, K):
    return [l[1:4] for l in P.gemm_plan(layout, M, N, K)[1]]


@pytest.mark.parametrize("M,N,K,tile", SMALLEST)
def test_products(M, N, K, tile):
    for layout in ("nn", "nt"):
        assert _tiles(layout, M, N, K) == [tile + (1,)]
    check_products(M, N, K, "nn", "nt")


@pytest.mark.parametrize("arch,hidden,ffn,mb,res32,fused,tile", [
    # GeLU and its derivative with the column sums behind it: the MLP matrices [hidden, ffn]
    ("gpt", 128, 6144, 6, 0, "fc1", (128, 192)), ("gpt", 256, 4096, 9, 0, "fc1", (192, 128)), ("gpt", 384, 5632, 15, 0, "fc1", (192, 256)),
    ("gpt", 2048, 2560, 26, 0, "fc1", (256, 160)), ("gpt", 2048, 6144, 12, 0, "fc1", (256, 192)),
    # residual adds: the output of the second matrix; SwiGLU and its derivative
    ("gpt", 4096, 256, 9, 0, "fc2", (192, 128)), ("llama", 4096, 256, 9, 1, "fc2", (192, 128)), ("llama", 256, 4096, 9, 0, "fc1", (192, 128)),
    ("llama", 128, 6144, 6, 0, "fc1", (128, 192)), ("llama", 2048, 2560, 26, 0, "fc1", (256, 160)),
    # the same adds where 48 or 40 lanes of a wave hold a piece: in 16 bits, and (res32) fp32 to fp32 in the first layer and to 16 bits in the second
    ("gpt", 6144, 128, 6, 0, "fc2", (128, 192)), ("llama", 6144, 128, 6, 1, "fc2", (128, 192)),
    ("gpt", 2560, 2048, 26, 0, "fc2", (256, 160)), ("gpt", 2560, 2048, 26, 1, "fc2", (256, 160))])
def test_epilogues(arch, hidden, ffn, mb, res32, fused, tile):
    """Gates: those of the stage parity tests (measured 3e-3 .. 8e-3, 2e-2 and 3e-2 allowed)."""
    T = mb * 128
    assert _tiles("nt" if fused == "fc1" else "nn", T, ffn if fused == "fc1" else hidden, hidden if fused == "fc1" else ffn) == [tile + (1,)]
    w = dict(arch=arch, n_layers=1 + res32, hidden=hidden, n_heads=2, head_dim=64, ffn=ffn, seq=128, mb=mb, n_mb=2, tp=1, recompute=0, res32=res32)
    gcfg, ocfg = U.make_cfgs(w, wgrad_group=2)
    params = [SI.draw_layer_params(w, l, perturb_vectors=True) for l in range(w["n_layers"])]
    xs, dys = ([SI.draw_activation(w, n, m) for m in range(2)] for n in ("x", "dy"))
    st = P.Stage(gcfg)
    U.load_params(st, params)
    ys, dxs = U.run_gpu(st, xs, dys)
    U.compare_stage(st, params, ys, dxs, *U.run_oracle(ocfg, params, xs, dys, np.float32))


@pytest.mark.parametrize("arch,hidden,ffn,grad", [("gpt", 4096, 256, "dc"), ("llama", 256, 4096, "du")])
def test_streams_change_no_bit(arch, hidden, ffn, grad, monkeypatch):
    """Input gradients that take 192 x 128 tiles by themselves, and 128 x 128 ones beside a second stream's weight gradients.  In the first
    stage also that of the output projection (k = 4096)."""
    T, heads = 1152, hidden // 128
    shapes = [(T, hidden, ffn), (T, hidden, hidden)] if grad == "dc" else [(T, ffn, hidden)]
    for shape in shapes:
        assert _tiles("nt", *shape) == [(192, 128, 1)]
    res = []
    for gflop in ("0", "1e9"):
        monkeypatch.setenv("AH_SIDE_STREAM_MIN_GFLOP", gflop)   # read when the stage is created
        st = P.Stage(P.StageConfig.make(arch=arch, n_layers=1, hidden=hidden, n_heads=heads, head_dim=128, ffn=ffn, seq=128, mb=9, n_mb=2))
        assert st.backward_streams() == (2 if gflop == "0" else 1)
        g = torch.Generator(device="cuda").manual_seed(9)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.03)
        out = []
        for _ in range(2):
            st.zero_grads()
            for _ in range(2):
                x, dy = (torch.randn(T, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
                y, dx = torch.empty_like(x), torch.empty_like(x)
                st.forward(0, x, y)
                st.backward(0, dy, dx)
                out += [y, dx]
            torch.cuda.synchronize()
            out.append(st.grads.clone())
        st.close()
        res.append(out)
    assert torch.isfinite(res[0][-1]).all() and all(torch.equal(a, b) for a, b in zip(*res))
