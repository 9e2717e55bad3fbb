"""GEMM entry points at the sizes where a tile shape begins, ends or leaves a remainder, against float64 products.

The launcher picks the tile by the output and k extents; the cases below reach every tile shape (64 x 64, 64 x 128 and,
for long k, 128 x 128 with the k axis split between waves, 128 x 128, the 256-wide ones), tile counts that are no multiple of the 8 XCDs,
and k extents from one ring fill less (k = 128 is two k-blocks, the ring holds three to five) to several.

Tolerance: a bf16 output is the fp32 sum rounded once, 2^-9 of its value at most (2^-8 between neighbouring values);
an fp32 sum of k products of N(0,1) values in any order is within 1e-6 sqrt(k) max|ref| here."""
import numpy as np
import pytest
import torch

import paper_2512_20953_amd as P

pytestmark = pytest.mark.gpu

SHAPES = [(128, 128, 128), (128, 384, 256), (384, 640, 384), (256, 256, 1024), (640, 1152, 640), (1024, 1024, 512), (896, 1152, 384),
          (1024, 2048, 128), (2048, 1024, 640), (1920, 1664, 256), (2048, 2048, 256), (2048, 2048, 4224), (2048, 2048, 5248), (1152, 4352, 128), (4096, 4096, 128)]


def _close(got, ref, k, bf16):
    tol = (2.0 ** -8) * ref.abs() * (1 if bf16 else 0) + 1e-6 * np.sqrt(k) * ref.abs().max()
    bad = (got.double() - ref).abs() > tol
    assert not bad.any(), "%d elements off, first at %s" % (int(bad.sum()), bad.nonzero()[0].tolist())


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_tiles(M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A, B, bias = rnd(M, K), rnd(K, N), rnd(N)
    ref = A.double() @ B.double()
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    P.gemm_nn(A, B, bias, C)
    _close(C, ref + bias.double(), K, True)
    C.fill_(float("nan"))
    P.gemm_nt(A, B.t().contiguous(), C)
    _close(C, ref, K, True)
    D0 = torch.randn(M, N, generator=g, device="cuda")
    D = D0.clone()
    P.gemm_tn(A.t().contiguous(), B, D, 1)
    _close(D, ref + D0.double(), K, False)
    half = K // 256 * 128
    if half:                                        # the k axis in two buffers of equal length
        At, Bh = A.t().contiguous()[:2 * half], B[:2 * half]
        P.gemm_tn_segmented([At[:half].clone(), At[half:].clone()], [Bh[:half].clone(), Bh[half:].clone()], D, 0)
        _close(D, At.double().t().contiguous() @ Bh.double(), K, False)
    if N % 256 == 0:                                # gate | up halves paired inside a tile
        U = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
        Mo = torch.empty(M, N // 2, dtype=torch.bfloat16, device="cuda")
        P.gemm_nn_swiglu(A, B, U, Mo)
        _close(U, ref, K, True)
        _close(Mo, torch.nn.functional.silu(ref[:, :N // 2]) * ref[:, N // 2:], K, True)


@pytest.mark.parametrize("arch,n_mb", [("gpt", 8), ("gpt", 11), ("llama", 7)])
def test_group_products_with_the_k_axis_shared_by_blocks(arch, n_mb):
    """Weight gradients of a narrow stage over groups of 8 micro-batches x 2048 tokens: 12 .. 64 tiles of 64 x 64, so
    the k axis is cut into shares of whole micro-batches (8, 4 or 2; an incomplete group of 3 or 7 into 3 or 7).
    Against the sums taken per micro-batch: the same up to the order of fp32 additions, y and dx bit for bit."""
    grads, outs = [], []
    for group in (1, 8):
        cfg = P.StageConfig.make(arch=arch, n_layers=2, hidden=256, n_heads=4, head_dim=64, ffn=512, seq=512, mb=4, n_mb=n_mb,
                                 max_in_flight=group, wgrad_group=group)
        st = P.Stage(cfg)
        g = torch.Generator(device="cuda").manual_seed(5)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.05)
        for repeat in range(2):                     # the second iteration adds to nothing of the first
            st.zero_grads()
            g.manual_seed(6)
            ys = []
            for m in range(n_mb):
                x, dy = (torch.randn(2048, 256, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
                y, dx = torch.empty_like(x), torch.empty_like(x)
                st.forward(m % group, x, y)
                st.backward(m % group, dy, dx)
                ys += [y, dx]
            st.flush_grads()
        torch.cuda.synchronize()
        grads.append([st.grad_view(l, n).clone() for l in range(2) for n in ("wqkv", "wo", "w1", "w2")])
        outs.append(ys)
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    for a, b in zip(*grads):
        assert ((a - b).double().norm() / a.double().norm()).item() <= 2e-6


@pytest.mark.parametrize("arch", ["gpt", "llama"])
@pytest.mark.parametrize("recompute", [0, 1])
def test_second_stream_by_size_changes_no_bit(arch, recompute, monkeypatch):
    """Whether the per-micro-batch weight gradients run on the second stream is decided by their flops; a small stage
    keeps one stream.  Forced either way: the same bits, over two iterations on the same stage."""
    res = []
    for gflop in ("0", "1e9"):
        monkeypatch.setenv("AH_SIDE_STREAM_MIN_GFLOP", gflop)   # read when the stage is created
        cfg = P.StageConfig.make(arch=arch, n_layers=3, hidden=256, n_heads=4, head_dim=64, ffn=512, seq=256, mb=2, n_mb=2, recompute=recompute)
        st = P.Stage(cfg)
        assert st.backward_streams() == (2 if gflop == "0" else 1)
        g = torch.Generator(device="cuda").manual_seed(9)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.05)
        out = []
        for it in range(2):
            st.zero_grads()
            for m in range(2):
                x, dy = (torch.randn(512, 256, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
                y, dx = torch.empty_like(x), torch.empty_like(x)
                st.forward(0, x, y)
                st.backward(0, dy, dx)
                out += [y, dx]
            torch.cuda.synchronize()
            out.append(st.grads.clone())
        res.append(out)
    assert all(torch.equal(a, b) for a, b in zip(*res))


@pytest.mark.parametrize("hidden,ffn", [(2048, 8192), (2048, 4224)])
def test_dx_depends_on_neither_streams_nor_groups(hidden, ffn, monkeypatch):
    """2048 x 2048 input gradients over k = 4224 .. 8192 (the longer ones' tile splits the k axis between its waves): with
    and without the second stream, and with the weight gradients of a group deferred or not, y and dx are the same bits."""
    res = []
    for group, gflop, defer, streams in ((1, "0", "1", 2), (1, "1e9", "1", 1), (2, "0", "1", 1), (2, "0", "0", 2)):
        monkeypatch.setenv("AH_SIDE_STREAM_MIN_GFLOP", gflop)   # both read when the stage is created
        monkeypatch.setenv("AH_DEFER_WGRADS", defer)
        cfg = P.StageConfig.make(arch="gpt", n_layers=1, hidden=hidden, n_heads=16, head_dim=128, ffn=ffn, seq=2048, mb=1, n_mb=2,
                                 max_in_flight=group, wgrad_group=group)
        st = P.Stage(cfg)
        assert st.backward_streams() == streams
        g = torch.Generator(device="cuda").manual_seed(9)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.02)
        st.zero_grads()
        out = []
        for m in range(2):
            x, dy = (torch.randn(2048, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
            y, dx = torch.empty_like(x), torch.empty_like(x)
            st.forward(m % group, x, y)
            st.backward(m % group, dy, dx)
            out += [y, dx]
        st.flush_grads()
        torch.cuda.synchronize()
        st.close()
        res.append(out)
    for other in res[1:]:
        assert all(torch.equal(a, b) for a, b in zip(res[0], other))


@pytest.mark.parametrize("rows,hidden,heads", [(128, 256, 1), (384, 640, 5), (4096, 1024, 8), (8192, 512, 4), (2048, 2048, 16)])
def test_rotary_epilogue_against_its_kernel(rows, hidden, heads, monkeypatch):
    """128-wide heads: where it pays, the QKV product takes tiles whose waves hold whole heads although others fit the
    output better, and rotates in its epilogue; the smallest outputs keep the separate rotary kernel.  Against that
    kernel, which rounds q and k once more: 2^-9 of their values, and no more than that on the scores, whose size is
    about 1 here; with the two roundings of the outputs, 2^-7 of the norm in all."""
    res = []
    for kernel in (False, True):
        if kernel:
            monkeypatch.setenv("AH_ROPE_KERNEL", "1")            # read when the stage is created
        seq = min(rows, 2048)
        cfg = P.StageConfig.make(arch="llama", n_layers=1, hidden=hidden, n_heads=heads, head_dim=128, ffn=512, seq=seq, mb=rows // seq, n_mb=1)
        st = P.Stage(cfg)
        g = torch.Generator(device="cuda").manual_seed(3)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * hidden ** -0.5)
        for name in ("ln1_g", "ln2_g"):
            st.param_view(0, name).fill_(1.0)
        x, dy = (torch.randn(rows, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
        y, dx = torch.empty_like(x), torch.empty_like(x)
        st.zero_grads()
        st.forward(0, x, y)
        st.backward(0, dy, dx)
        torch.cuda.synchronize()
        res.append([t.double() for t in (y, dx, st.grad_view(0, "wqkv"))])
        st.close()
    for a, b in zip(*res):
        assert torch.isfinite(a).all() and ((a - b).norm() / b.norm()).item() <= 2.0 ** -7
