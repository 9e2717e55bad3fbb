"""GEMM entry points at the sizes where a tile shape begins, ends or leaves a remainder, against float64 products.

The launcher picks the tiles by the output and k extents.  SHAPES are small outputs: tile counts that are no multiple of
the 8 XCDs, and k extents from less than one ring fill (k = 128 is two k-blocks, the ring holds three to five) to several.
COVERS are the smallest products found for every tile shape of every layout and for outputs covered by two launches; each
asserts the cover it is there for.

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


# (rows, columns, waves that split a k-block) of the tiles of each launch
T64, T64x128, T128, T128K = (64, 64, 4), (64, 128, 2), (128, 128, 1), (128, 128, 4)
T128x256, T256x128, T256 = (128, 256, 1), (256, 128, 1), (256, 256, 1)
COVERS = [
    # forward (with the SwiGLU form of it: N is a multiple of 256 but for 256 x 128, which no such small output takes) ..
    ("nn", 128, 256, 128, [T64]), ("nn", 128, 4352, 128, [T64x128]), ("nn", 640, 3328, 128, [T128]), ("nn", 640, 3328, 5248, [T128K]),
    ("nn", 1280, 3328, 2048, [T128x256]), ("nn", 2560, 1664, 2048, [T256x128]), ("nn", 3328, 3840, 384, [T256]),
    ("nn", 1664, 5120, 2048, [T64, T128x256]), ("nn", 3328, 5120, 1024, [T64, T256]), ("nn", 5120, 3328, 2048, [T64x128, T256]),
    ("nn", 3840, 2304, 5248, [T64, T256x128]),
    # .. input gradient ..
    ("nt", 128, 128, 128, [T64]), ("nt", 640, 896, 128, [T64x128]), ("nt", 1280, 1664, 128, [T128]), ("nt", 1280, 1664, 5248, [T128K]),
    ("nt", 1664, 2560, 2048, [T128x256]), ("nt", 2560, 1664, 2048, [T256x128]), ("nt", 3328, 3840, 384, [T256]),
    ("nt", 2560, 1664, 5248, [T64, T128K]), ("nt", 1664, 5120, 2048, [T64, T128x256]), ("nt", 5120, 3328, 2048, [T64x128, T256]),
    # .. weight gradient
    ("tn", 128, 128, 128, [T64]), ("tn", 640, 1664, 128, [T64x128]), ("tn", 1280, 1664, 128, [T128]), ("tn", 1664, 2560, 128, [T128x256]),
    ("tn", 2560, 1664, 512, [T256x128]), ("tn", 2560, 3328, 128, [T256]), ("tn", 3328, 5120, 256, [T64, T256]),
    ("tn", 5120, 3328, 384, [T64x128, T256]), ("tn", 5120, 3584, 512, [T128, T256]), ("tn", 1664, 5120, 2048, [T64, T128x256]),
]


@pytest.mark.parametrize("layout,M,N,K,cover", COVERS)
def test_every_tile_and_cover(layout, M, N, K, cover):
    shares, launches = P.gemm_plan(layout, M, N, K)
    assert shares == 1 and [l[1:4] for l in launches] == cover
    check_products(M, N, K, layout)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_tiles(M, N, K):
    check_products(M, N, K, "nn", "nt", "tn")


def check_products(M, N, K, *layouts):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    A, B, bias = rnd(M, K), rnd(K, N), rnd(N)
    ref = A.double() @ B.double()
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    if "nn" in layouts:
        P.gemm_nn(A, B, bias, C)
        _close(C, ref + bias.double(), K, True)
        if N % 256 == 0:                                # gate | up halves paired inside a tile
            U = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
            Mo = torch.full((M, N // 2), float("nan"), dtype=torch.bfloat16, device="cuda")
            P.gemm_nn_swiglu(A, B, U, Mo)
            _close(U, ref, K, True)
            _close(Mo, torch.nn.functional.silu(ref[:, :N // 2]) * ref[:, N // 2:], K, True)
    if "nt" in layouts:
        C.fill_(float("nan"))
        P.gemm_nt(A, B.t().contiguous(), C)
        _close(C, ref, K, True)
    if "tn" in layouts:
        At = A.t().contiguous()
        D0 = torch.randn(M, N, generator=g, device="cuda")
        D = D0.clone()
        P.gemm_tn(At, B, D, 1)
        _close(D, ref + D0.double(), K, False)
        D.fill_(float("nan"))
        P.gemm_tn(At, B, D, 0)
        _close(D, ref, K, False)
        half = K // 256 * 128
        if half:                                        # the k axis in two buffers of equal length
            At, Bh = At[:2 * half], B[:2 * half]
            P.gemm_tn_segmented([At[:half].clone(), At[half:].clone()], [Bh[:half].clone(), Bh[half:].clone()], D, 0)
            _close(D, At.double().t().contiguous() @ Bh.double(), K, False)


# (n_seg pending micro-batches, matrix) -> (shares, tile): what the case is there for
SHARES = [
    # 12 .. 64 tiles of 64 x 64: whole micro-batches per share (8; an incomplete group of 3 or 7 into 3 or 7)
    ("gpt", 256, 64, 512, 512, 4, 8, 8, {(8, "w1"): (8, T64), (8, "wqkv"): (8, T64x128)}),
    ("gpt", 256, 64, 512, 512, 4, 11, 8, {(3, "w1"): (3, T64), (3, "wqkv"): (3, T64)}),
    ("llama", 256, 64, 512, 512, 4, 7, 8, {(7, "wqkv"): (7, T64x128)}),
    # the large tiles' pipeline: two micro-batches per share (the buffers change inside it), one, and, of an incomplete
    # group of five, one
    ("gpt", 1024, 64, 4096, 512, 8, 13, 8, {(8, "w1"): (4, T256), (8, "w2"): (4, T256), (8, "wqkv"): (4, T256), (8, "wo"): (8, T128x256),
                                            (5, "wqkv"): (5, T256)}),
    ("gpt", 768, 64, 3072, 512, 8, 11, 8, {(8, "wqkv"): (4, T128x256), (8, "w1"): (4, T256), (3, "w1"): (3, T128x256), (3, "wo"): (3, T64x128)}),
    ("gpt", 512, 64, 2048, 512, 4, 8, 8, {(8, "w1"): (4, T128), (8, "wo"): (8, T64x128), (8, "wqkv"): (8, T128x256)}),
    ("gpt", 384, 64, 2816, 1024, 1, 7, 7, {(7, "w2"): (7, T256x128)}),
    # one pending micro-batch, its k axis cut inside the one piece: both pipelines
    ("gpt", 512, 64, 512, 1024, 8, 5, 4, {(1, "wqkv"): (4, T128), (1, "w1"): (4, T64)}),
]


@pytest.mark.parametrize("arch,hidden,head_dim,ffn,seq,mb,n_mb,group,expect", SHARES)
def test_group_products_with_the_k_axis_shared_by_blocks(arch, hidden, head_dim, ffn, seq, mb, n_mb, group, expect, monkeypatch):
    """Deferred weight gradients whose outputs have fewer tiles than the chip has CUs: launched one by one, their k axis is cut into
    shares (`expect`).  Most of these groups go out as one launch instead; the same cases with AH_GEMM_SEPARATE set, where the
    shares run, are in test_gpu_grouped_wgrads.py.
    Against the sums taken per micro-batch: the same up to the order of fp32 additions (2e-6 of the norm over the 32768
    tokens of the full-size comparison; a sum's rounding errors grow with the square root of its length), y and dx bit for bit."""
    monkeypatch.setenv("AH_DEFER_WGRADS", "1")
    T = mb * seq
    matrices = {"w2": (ffn, hidden), "w1": (hidden, (2 if arch == "llama" else 1) * ffn), "wo": (hidden, hidden), "wqkv": (hidden, 3 * hidden)}
    full = {n: P.gemm_plan("tn", *s, T * group, group, s[0] * s[1] * 16)[0] for n, s in matrices.items()}
    room = max(s[0] * s[1] * full[n] for n, s in matrices.items() if full[n] > 1)       # the stage's buffer for partial sums
    for (n_seg, name), (shares, tile) in expect.items():
        got = P.gemm_plan("tn", *matrices[name], T * n_seg, n_seg, room)
        assert (got[0], [l[1:4] for l in got[1]]) == (shares, [tile]), (n_seg, name)
    grads, outs = [], []
    for G in (1, group):
        cfg = P.StageConfig.make(arch=arch, n_layers=2, hidden=hidden, n_heads=hidden // head_dim, head_dim=head_dim, ffn=ffn, seq=seq, mb=mb,
                                 n_mb=n_mb, max_in_flight=G, wgrad_group=G)
        st = P.Stage(cfg)
        g = torch.Generator(device="cuda").manual_seed(5)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.8 * hidden ** -0.5)
        for repeat in range(2):                     # the second iteration adds to nothing of the first
            st.zero_grads()
            g.manual_seed(6)
            ys = []
            for m in range(n_mb):
                x, dy = (torch.randn(T, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
                y, dx = torch.empty_like(x), torch.empty_like(x)
                st.forward(m % G, x, y)
                st.backward(m % G, dy, dx)
                ys += [y, dx]
            st.flush_grads()
        torch.cuda.synchronize()
        grads.append([st.grad_view(l, n).clone() for l in range(2) for n in ("wqkv", "wo", "w1", "w2")])
        outs.append(ys)
        st.close()
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    for a, b in zip(*grads):
        assert ((a - b).double().norm() / a.double().norm()).item() <= 2e-6 * max(1.0, T * n_mb / 32768) ** 0.5


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
    assert [P.gemm_plan("nt", 2048, hidden, k)[1][0][1:4] for k in (ffn, 3 * hidden)] == [T128K if ffn > 5120 else T128, T128K]
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
