"""GPU parity of stages at the widths and row counts where the LayerNorm kernels change their shape: 16, 32 and 64 lanes a row, one to
eight chunks of columns, the last of them full, partly empty or a single group of lanes, and rows that do not fill a workgroup."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["unet", "dit"])
@pytest.mark.parametrize("batch,tokens,heads,d_head", [
    (65, 256, 1, 40),      # 16 lanes, part of one chunk
    (67, 251, 4, 64),      # 16 lanes, four whole chunks, ragged rows
    (64, 257, 9, 40),      # 16 lanes, six chunks, the last partly empty
    (33, 249, 5, 80),      # 32 lanes, 400 columns
    (32, 257, 8, 96),      # 32 lanes, 768 columns
    (3, 5, 1, 8),          # less than a group of lanes
    (2, 7, 14, 24),        # few rows: 64 lanes, 336 columns
    (1, 9, 23, 88),        # 64 lanes, eight chunks, 2024 columns
])
def test_layernorm_shapes(kind, batch, tokens, heads, d_head):
    import torch
    from paper_2405_01248_amd.harness import DeviceStage
    from test_gpu_parity import _compare, _oracle_stage
    d, ctx = heads * d_head, (0, 0) if kind == "dit" else (4, 8)
    cfg = si.StageConfig("ln_" + kind, si.DIT if kind == "dit" else si.UNET, "bf16", 1, batch, tokens, d, heads, d_head, *ctx, 32, 1e-6 if kind == "dit" else 1e-5, int(kind == "dit"))
    inp = si.make_stage_inputs(cfg, seed=5)
    ds = DeviceStage(cfg, inp)
    ds.step()
    torch.cuda.synchronize()
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))


@pytest.mark.parametrize("mode", [1, 2])
def test_rows_of_an_encoder_do_not_depend_on_their_number(mode):
    # 128 samples of 77 rows are more than the lanes' shape for few rows takes in a stage, one sample is not
    import numpy as np
    import torch
    from paper_2405_01248_amd.harness import DeviceEncoder
    cfg = si.EncoderConfig("ln_enc", "bf16", 1, 512, 8, 64, 77, 256, 512, 128)
    de = DeviceEncoder(cfg, si.make_encoder_inputs(cfg, seed=2))
    de.enc.set_batch_invariant(mode)
    de.ws = torch.empty(de.enc.workspace_bytes(de.gb), dtype=torch.uint8, device=de.device)
    outs = []
    for b in (128, 1):
        de.hidden.zero_()
        de.run_slices(b)
        torch.cuda.synchronize()
        outs.append(de.output())
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("kind,batch,tokens,heads,d_head,part", [
    ("dit", 56, 256, 18, 64, 8),       # rows of 1152: 768 workgroups at a time, 20 rows each; the slices 4
    ("dit", 9, 1024, 20, 80, 1),       # rows of 1600: 512, 20 rows, the last of a sample with 4
    ("dit", 2, 5003, 24, 64, 1),       # rows of 1536, ragged samples: 20 rows and 16
    ("unet", 14, 1024, 20, 80, 2),     # rows of 1600: 768, 20 rows
])
def test_wide_rows_in_one_round_of_workgroups(kind, batch, tokens, heads, d_head, part):
    """Gradients of a micro-batch whose LayerNorm backward takes more rows a workgroup are the sum of its slices', which take few."""
    import numpy as np
    import torch
    from paper_2405_01248_amd.harness import DeviceStage, rel_l2
    d, ctx = heads * d_head, (0, 0) if kind == "dit" else (4, 8)
    cfg = si.StageConfig("ln_wide", si.DIT if kind == "dit" else si.UNET, "bf16", 2 if kind == "dit" else 1, batch, tokens, d, heads, d_head, *ctx, 32, 1e-6 if kind == "dit" else 1e-5, int(kind == "dit"))
    inp = si.make_stage_inputs(cfg, seed=7)

    def run(lo, hi):
        per_sample = ("x", "dy", "x_sc", "ctx", "cond")
        ds = DeviceStage(cfg.replace(batch=hi - lo), {k: v[lo:hi] if k in per_sample else v for k, v in inp.items()})
        ds.step()
        torch.cuda.synchronize()
        return ds.results()

    whole = run(0, batch)
    sums, worst = {}, {}
    for lo in range(0, batch, part):
        r = run(lo, lo + part)
        for k in ("y", "dx") + (("dcond",) if kind == "dit" else ()):
            worst[k] = max(worst.get(k, 0.0), rel_l2(whole[k][lo:lo + part], r[k]))
        for k, g in r["grads"].items():
            sums[k] = sums.get(k, 0.0) + g.astype(np.float64)
    for k, g in sums.items():
        worst[k] = rel_l2(whole["grads"][k], g)
    # the same operands and roundings to bf16, tiles with other orders of addition in between: 2^-9 of a value where one rounds the other way
    assert max(worst.values()) <= 2.0 ** -9, {k: v for k, v in worst.items() if v > 2.0 ** -10}
