"""The workspace holds room for partial sums of weight gradients only where a group's products can still cut their k axis into shares."""
import pytest

import paper_2512_20953_amd as P
from paper_2512_20953_amd.binding import query_sizes


def _workspace(arch, hidden, heads, head_dim, ffn, seq, mb, group):
    cfg = P.StageConfig.make(arch=arch, n_layers=1, hidden=hidden, n_heads=heads, head_dim=head_dim, ffn=ffn, seq=seq, mb=mb, max_in_flight=group,
                             wgrad_group=group)
    return query_sizes(cfg)["workspace_bytes"]


@pytest.mark.parametrize("stage,one_by_one", [
    # (bytes of partial sums with the products one by one); in one launch, as every group of these goes out, full or not, none
    (("bert", 1024, 16, 64, 4096, 512, 8, 8), 64 << 20),
    (("gpt", 768, 12, 64, 3072, 512, 8, 8), 36 << 20),
    (("gpt", 512, 8, 64, 2048, 512, 4, 8), 24 << 20),
    (("gpt", 2048, 16, 128, 8192, 2048, 1, 16), 64 << 20),
])
def test_no_room_for_shares_that_never_run(stage, one_by_one, monkeypatch):
    monkeypatch.setenv("AH_DEFER_WGRADS", "0")
    without = _workspace(*stage)
    monkeypatch.setenv("AH_DEFER_WGRADS", "1")
    assert _workspace(*stage) == without
    monkeypatch.setenv("AH_GEMM_SEPARATE", "1")
    assert _workspace(*stage) == without + one_by_one
