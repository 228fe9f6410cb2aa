"""fp32 U-Net blocks, whose projections normalise their rows themselves up to 256 columns, against the fp64 oracle (result, gradients, and with them what the
LayerNorms keep for the backward): rows that end inside a tile, one row, the narrowest, both sides of the widths where four waves become eight (128) and where a
LayerNorm launch takes over (256).  Metric per tensor: max|gpu - oracle| / max|oracle| <= 1e-4, the bar of the other fp32 stages: sums of at most 4 * 272 terms over
two blocks, each term and each sum rounded to 2^-24."""
import pytest

import synth_inputs as si
from test_gpu_parity import _compare, _oracle_stage, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,tokens", [(1, 1), (1, 33), (2, 32)])
@pytest.mark.parametrize("heads,d_head", [(1, 16), (5, 16), (4, 32), (9, 16), (8, 32), (17, 16)])
def test_layer_norm_inside_the_fp32_projections(heads, d_head, batch, tokens):
    d = heads * d_head
    cfg = si.StageConfig(f"norm_f32_{d}_{batch}x{tokens}", si.UNET, "f32", 2, batch, tokens, d, heads, d_head, 5, 24, 4 * d)
    ds, inp = _run(cfg, seed=d + tokens)
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))
