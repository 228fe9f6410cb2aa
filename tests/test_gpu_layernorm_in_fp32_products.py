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


def _launches(ds):
    import torch
    from paper_2405_01248_amd import binding as B
    B.ktime_begin(256)
    ds.stage.fwd(ds.params, ds.x, ds.cc, ds.y, ds.ws, True)
    kinds = [r["kind"] for r in B.ktime_end(256)]
    torch.cuda.synchronize()
    return {k: kinds.count(k) for k in ("ln_fwd", "gemm_f32")}


@pytest.mark.parametrize("batch,tokens", [(1, 33), (2, 45)])
@pytest.mark.parametrize("heads,d_head", [(9, 16), (16, 16)])
@pytest.mark.parametrize("ctx_tokens,ctx_dim", [(5, 136), (37, 272)])
def test_the_context_projection_beside_a_normalising_one_of_eight_waves(heads, d_head, batch, tokens, ctx_tokens, ctx_dim):
    # widths and context widths above 128 share a launch and its LDS; a context of 24 has one of its own
    d = heads * d_head
    cfg = si.StageConfig(f"norm_f32_ctx_{d}_{ctx_dim}", si.UNET, "f32", 2, batch, tokens, d, heads, d_head, ctx_tokens, ctx_dim, 4 * d)
    ds, inp = _run(cfg, seed=d + ctx_dim)
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))
    narrow, _ = _run(cfg.replace(ctx_dim=24), seed=1)
    assert _launches(ds)["gemm_f32"] == _launches(narrow)["gemm_f32"] - cfg.n_blocks


@pytest.mark.parametrize("batch,launches", [(256, 0), (257, 1)])
def test_the_line_between_the_product_and_a_launch(batch, launches):
    # 64 columns: the feed-forward's 16 column tiles by 256 row tiles are the 4096 up to which the product normalises its rows
    cfg = si.StageConfig(f"norm_f32_line_{batch}", si.UNET, "f32", 1, batch, 32, 64, 4, 16, 4, 24, 256)
    ds, inp = _run(cfg, seed=batch)
    assert _launches(ds)["ln_fwd"] == launches
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))


@pytest.mark.parametrize("heads", [4, 12])
def test_infinities_and_nan_stay_in_their_sample(heads):
    import torch
    d = 16 * heads
    cfg = si.StageConfig(f"norm_f32_nan_{d}", si.UNET, "f32", 1, 3, 45, d, heads, 16, 5, 24, 4 * d)
    ds, _ = _run(cfg, seed=d)
    clean = ds.y.clone()
    ds.x[0, 3, 5], ds.x[2, 44, d - 1] = float("nan"), float("inf")
    ds.stage.fwd(ds.params, ds.x, ds.cc, ds.y, ds.ws, True)
    torch.cuda.synchronize()
    assert torch.equal(ds.y[1], clean[1]) and ds.y[0].isnan().all() and ds.y[2].isnan().all()
