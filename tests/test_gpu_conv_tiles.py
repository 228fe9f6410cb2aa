"""The convolution's kernel for eight input channels and its tiles for few pixels (64 x 64 and 128 x 128) at the edges of their range, against the fp64 oracle
through the image encoder's C ABI: pixel counts around a tile, a single pixel, the 8-channel head, stride 2, GroupNorm sums over
blocks of 64 pixels.  Metric: max|gpu - oracle| / max|oracle| <= 2e-2 (bf16 storage)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import image_encoder as ie

pytestmark = pytest.mark.gpu


def _layer(kind, ci, co, stride, hw, batch, groups=8):
    return si.ImageEncoderConfig(f"few_px_{kind}_{ci}_{co}_s{stride}_{hw[0]}x{hw[1]}_{batch}", "bf16", hw[0], hw[1], ci, groups,
                                 ((kind, ci, co, stride),), batch)


@pytest.mark.parametrize("cfg", [
    _layer("conv", 64, 64, 1, (1, 1), 1),
    _layer("conv", 128, 8, 1, (9, 7), 3),            # 63 pixels a sample, 8 of 64 channels
    _layer("conv", 512, 72, 1, (5, 13), 1),          # 65 pixels, two channel tiles
    _layer("conv", 64, 128, 2, (31, 34), 2),
    _layer("resnet", 64, 64, 1, (8, 8), 3),          # one statistics block a sample
    _layer("resnet", 128, 136, 1, (24, 24), 2),      # nine blocks of 64, three channel tiles
    _layer("conv", 8, 8, 1, (3, 5), 2),              # eight input channels: less than a band of pixels
    _layer("conv", 8, 72, 2, (33, 31), 3),           # ... ragged bands and channels, stride 2
    _layer("resnet", 8, 64, 1, (24, 24), 3),         # ... statistics blocks of 64, nine a sample
    _layer("resnet", 8, 128, 1, (128, 132), 1),      # ... statistics blocks of 256
    _layer("resnet", 64, 64, 1, (45, 45), 2, 4),     # 16 channels a group, 4050 of 4096 values in the one-launch GroupNorm
    _layer("resnet", 64, 128, 1, (7, 5), 2, 2),      # ... 32 and 64 channels a group
    _layer("resnet", 256, 256, 1, (64, 80), 1, 32),  # enough tiles for the 128-row shape
], ids=lambda c: c.name)
def test_few_pixel_tiles_match_oracle(cfg):
    import torch
    from paper_2405_01248_amd.harness import DeviceImageEncoder, rel_err
    inp = si.make_image_encoder_inputs(cfg, seed=3, randomize_norm=True, weight_std=0.0)
    ref = ie.encoder_fwd_partial(inp["params"], cfg.layer_dicts(), inp["x"], 0, 1, 0, cfg.global_batch, cfg.groups, cfg.gn_eps)
    de = DeviceImageEncoder(cfg, inp)
    de.run_slices(cfg.global_batch)
    torch.cuda.synchronize()
    whole = de.output()
    assert rel_err(whole, ref) <= 2e-2
    de.out.zero_()
    de.run_slices(1)
    torch.cuda.synchronize()
    assert np.array_equal(de.output(), whole)


@pytest.mark.parametrize("hw,c,batch", [((8, 8), 64, 5), ((40, 32), 72, 4), ((56, 46), 128, 2), ((66, 64), 64, 2)],
                         ids=["one_by_one", "one_launch_ragged", "softmax_2576", "softmax_beyond_4096"])
def test_attention_of_several_samples_matches_oracle(hw, c, batch):
    """The attention block's products of a call's samples in one launch or one by one, and its softmax by row length: against
    the oracle, and the same bits one sample at a time."""
    import torch
    from paper_2405_01248_amd.harness import DeviceImageEncoder, rel_err
    cfg = _layer("attn", c, c, 1, hw, batch)
    inp = si.make_image_encoder_inputs(cfg, seed=4, randomize_norm=True, weight_std=0.0)
    ref = ie.encoder_fwd_partial(inp["params"], cfg.layer_dicts(), inp["x"], 0, 1, 0, cfg.global_batch, cfg.groups, cfg.gn_eps)
    de = DeviceImageEncoder(cfg, inp)
    de.run_slices(batch)
    torch.cuda.synchronize()
    whole = de.output()
    assert rel_err(whole, ref) <= 2e-2
    de.out.zero_()
    de.run_slices(1)
    torch.cuda.synchronize()
    assert np.array_equal(de.output(), whole)
