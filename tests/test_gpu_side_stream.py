"""The side stream of a stage (three and more blocks): results do not depend on whether it is used, nor on whether the forward
keeps its activations; buffers that consecutive blocks take in turn come round from the fourth block on."""
import numpy as np
import pytest

import synth_inputs as si
from test_gpu_parity import _compare, _oracle_stage, _run, test_step_can_be_captured_in_a_hip_graph_and_replayed as capture_and_replay

pytestmark = pytest.mark.gpu

FIVE_UNET = si.StageConfig("five_unet_bf16", si.UNET, "bf16", 5, 2, 200, 192, 3, 64, 77, 64, 288)
FIVE_DIT = si.StageConfig("five_dit_bf16", si.DIT, "bf16", 5, 3, 72, 144, 2, 72, 0, 0, 296, 1e-6, 1)
# few context rows and a long contraction: the K/V projection is cut along the contraction where it has scratch for it
WIDE_CTX = si.StageConfig("unet_wide_context", si.UNET, "bf16", 3, 1, 1024, 256, 4, 64, 77, 4096, 1024)


@pytest.mark.parametrize("cfg", [FIVE_UNET, FIVE_DIT], ids=lambda c: c.name)
def test_five_blocks_match_oracle(cfg):
    ds, inp = _run(cfg, randomize_ln=True)
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))


@pytest.mark.parametrize("cfg", [FIVE_UNET, FIVE_DIT, WIDE_CTX], ids=lambda c: c.name)
def test_overlap_and_saving_change_no_bit(cfg):
    import torch
    ds, _ = _run(cfg, randomize_ln=True)
    on = ds.results()
    ds.stage.set_overlap(False)
    ds.step()
    ds.stage.fwd(ds.params, ds.x, ds.cc, ds.y_sc, ds.ws_nograd, False)
    torch.cuda.synchronize()
    off = ds.results()
    assert np.array_equal(on["y"], off["y_sc"])
    for k in ("y", "dx"):
        assert np.array_equal(on[k], off[k]), k
    for k in on["grads"]:
        assert np.array_equal(on["grads"][k], off["grads"][k]), k


def test_five_blocks_in_a_graph():
    capture_and_replay(FIVE_UNET)


@pytest.mark.parametrize("cfg", [FIVE_UNET, FIVE_DIT, FIVE_DIT.replace(name="two_dit_bf16", n_blocks=2), FIVE_DIT.replace(name="dit_batch49", batch=49, tokens=5)],
                         ids=lambda c: c.name)
def test_profile_times_the_kernels_of_the_step(cfg):
    import torch
    from paper_2405_01248_amd import binding as B
    ds, _ = _run(cfg)
    launches = []
    for run in (lambda: ds.step(self_cond=False),
                lambda: ds.stage.profile(ds.params, ds.x, ds.cc, ds.y, ds.dy, ds.dx, ds.d_cond, ds.dparams, ds.ws, reps=1)):
        B.ktime_begin(4096)
        run()
        torch.cuda.synchronize()
        launches.append(sorted((r["kind"], r["m"], r["n"], r["k"]) for r in B.ktime_end(4096)))
    assert launches[0] == launches[1]


def test_timed_bytes_of_the_gated_branches():
    # beside gradient, input, residual gradient and result a LayerNorm backward moves the gated branch it serves; the last block's has a kernel of its own
    import torch
    from paper_2405_01248_amd import binding as B
    cfg = FIVE_DIT.replace(name="two_dit_bf16", n_blocks=2)
    ds, _ = _run(cfg)
    B.ktime_begin(4096)
    ds.step()
    torch.cuda.synchronize()
    rows = B.ktime_end(4096)
    t, d = cfg.batch * cfg.tokens, cfg.d_model
    assert sorted(r["bytes"] for r in rows if r["kind"] == "ln_bwd") == [12 * t * d + 8 * t] + 3 * [18 * t * d + 8 * t]
    assert sum(r["kind"] == "other" and (r["m"], r["n"]) == (t, d) and r["bytes"] == 8 * t * d for r in rows) == 1
