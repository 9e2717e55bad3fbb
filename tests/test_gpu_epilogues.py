"""The GeLU epilogues on each large tile, against the oracle: one GPT layer whose first MLP product and whose second one's input
gradient take that tile (asserted).  Their pieces run in a loop, and in backward the pre-activation passes through LDS two
strips of rows at a time.  Two micro-batches in one group, so that the column sums for the bias gradient are written and
added to.  Gates: those of the stage parity tests (a layer of bf16 tensors: 3e-3 .. 8e-3 measured, 2e-2 and 3e-2 allowed; the
pre-activation's bias gradient is compared like every other tensor)."""
import numpy as np
import pytest

import paper_2512_20953_amd as P
from synth import stage_inputs as SI
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [(4, 4224, 256, (128, 128)), (8, 4352, 1536, (128, 256)), (8, 4224, 2048, (256, 128)), (20, 5120, 384, (256, 256))]


@pytest.mark.parametrize("mb,ffn,hidden,tile", CASES)
def test_gelu_epilogues_on_every_large_tile(mb, ffn, hidden, tile):
    for layout in ("nn", "nt"):
        _, launches = P.gemm_plan(layout, mb * 128, ffn, hidden)
        assert [l[1:4] for l in launches] == [tile + (1,)]
    w = dict(arch="gpt", n_layers=1, hidden=hidden, n_heads=hidden // 128, head_dim=128, ffn=ffn, seq=128, mb=mb, n_mb=2, tp=1, recompute=0)
    gcfg, ocfg = U.make_cfgs(w, wgrad_group=2)
    params = [SI.draw_layer_params(w, 0, perturb_vectors=True)]
    xs, dys = ([SI.draw_activation(w, n, m) for m in range(2)] for n in ("x", "dy"))
    st = P.Stage(gcfg)
    U.load_params(st, params)
    ys, dxs = U.run_gpu(st, xs, dys)
    U.compare_stage(st, params, ys, dxs, *U.run_oracle(ocfg, params, xs, dys, np.float32))
