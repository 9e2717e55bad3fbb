"""Weight gradients of a layer in one launch: every tile the rule chooses, beside the products one by one."""
import pytest
import torch

import paper_2512_20953_amd as P
from tests.test_gpu_gemm_tiles import SHARES, test_group_products_with_the_k_axis_shared_by_blocks as products_one_by_one

pytestmark = pytest.mark.gpu

# arch, layers, hidden, heads, head_dim, ffn, seq, mb, micro-batches, group, recompute.  Groups run all four products together
# (in the last group of a case without a full one, over fewer micro-batches), single micro-batches two and two
CASES = [
    ("gpt", 2, 256, 4, 64, 1024, 128, 2, 4, 2, 0),     # 64 x 64 tiles, the first iteration overwrites, the second group adds
    ("gpt", 1, 640, 5, 128, 1152, 128, 3, 2, 1, 0),    # pairs of 384 tokens, which only tiles of up to 128 rows divide
    ("llama", 2, 384, 3, 128, 1408, 128, 1, 3, 1, 1),  # pairs over one k tile, recomputed forward
    ("llama", 1, 512, 8, 64, 1536, 256, 4, 5, 3, 0),   # an incomplete group of two
    ("llama", 1, 768, 12, 64, 1664, 128, 1, 2, 2, 0),  # 128 x 256 tiles
    ("gpt", 1, 768, 12, 64, 1536, 512, 4, 8, 8, 0),    # 256 x 128
    ("bert", 1, 1024, 16, 64, 4096, 512, 8, 3, 3, 0),  # 192 tiles of 256 x 256
    ("gpt", 1, 2048, 16, 128, 8192, 256, 4, 2, 2, 0),  # three whole rounds of them
]


@pytest.mark.parametrize("arch,layers,hidden,heads,head_dim,ffn,seq,mb,n_mb,group,recompute", CASES)
def test_layer_products_in_one_launch(arch, layers, hidden, heads, head_dim, ffn, seq, mb, n_mb, group, recompute, monkeypatch):
    """The same sums in another order: 2e-6 of the norm over 32768 tokens, growing with the square root of their number, as
    for any other tile; y and dx bit for bit.  Traced, so that what was launched is known."""
    monkeypatch.setenv("AH_DEFER_WGRADS", "1")
    T, res = mb * seq, []
    for separate in (True, False):
        if separate:
            monkeypatch.setenv("AH_GEMM_SEPARATE", "1")
        else:
            monkeypatch.delenv("AH_GEMM_SEPARATE")
        cfg = P.StageConfig.make(arch=arch, n_layers=layers, hidden=hidden, n_heads=heads, head_dim=head_dim, ffn=ffn, seq=seq, mb=mb,
                                 n_mb=n_mb, max_in_flight=group, wgrad_group=group, recompute=recompute)
        st = P.Stage(cfg)
        g = torch.Generator(device="cuda").manual_seed(5)
        st.params.copy_(torch.randn(st.params.shape, generator=g, device="cuda") * 0.8 * hidden ** -0.5)
        for repeat in range(2):
            st.zero_grads()
            g.manual_seed(6)
            st.trace_begin()
            ys = []
            for m in range(n_mb):
                x, dy = (torch.randn(T, hidden, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
                y, dx = torch.empty_like(x), torch.empty_like(x)
                st.forward(m % group, x, y)
                st.backward(m % group, dy, dx)
                ys += [y, dx]
            st.flush_grads()
            sites = {s["name"]: s["launches"] for s in st.trace_end()}
        wgrads = {n: k for n, k in sites.items() if "wgrad" in n}
        groups = -(-n_mb // group)
        if separate:
            assert set(wgrads) == {"gemm_tn.%s_wgrad" % n for n in ("fc2", "fc1", "wo", "qkv")}
        elif group > 1:
            assert wgrads == {"gemm_tn.layer_wgrads": groups * layers}
        else:
            assert wgrads == {"gemm_tn.mlp_wgrads": groups * layers, "gemm_tn.attn_wgrads": groups * layers}
        res.append((ys, [st.grad_view(l, n).clone() for l in range(layers) for n in ("wqkv", "wo", "w1", "w2")]))
        st.close()
    assert all(torch.equal(a, b) for a, b in zip(res[0][0], res[1][0]))
    for a, b in zip(res[0][1], res[1][1]):
        assert ((a - b).double().norm() / a.double().norm()).item() <= 2e-6 * max(1.0, T * n_mb / 32768) ** 0.5


@pytest.mark.parametrize("case", SHARES)
def test_k_shares_where_products_run_one_by_one(case, monkeypatch):
    """The shapes whose products, one by one, cut their k axis between blocks are together mostly enough for one launch."""
    monkeypatch.setenv("AH_GEMM_SEPARATE", "1")
    products_one_by_one(*case, monkeypatch)
