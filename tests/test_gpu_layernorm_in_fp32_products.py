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


@pytest.mark.parametrize("heads,d_head", [(4, 32), (9, 16), (8, 32), (17, 16)])
def test_switching_the_geglu_fusion_off_changes_no_bit(heads, d_head):
    # the third LayerNorm stands before the fused product and before the plain one: both add up its rows in the same order, with four waves and with eight
    import numpy as np
    import torch
    d = heads * d_head
    cfg = si.StageConfig(f"norm_f32_unfused_{d}", si.UNET, "f32", 2, 1, 45, d, heads, d_head, 5, 24, 4 * d)
    ds, _ = _run(cfg, seed=d)
    fused = ds.results()
    ds.stage.set_fusion(0)
    ds.step()
    torch.cuda.synchronize()
    plain = ds.results()
    assert np.array_equal(fused["y"], plain["y"]) and np.array_equal(fused["dx"], plain["dx"])
    assert all(np.array_equal(fused["grads"][k], plain["grads"][k]) for k in plain["grads"])
