"""Text-encoder calls of few rows, whose projections normalise their rows themselves (widths of 256 to 1024 that are multiples of 256, 32-row tiles, one a CU at
most), against the fp64 oracle: rows that end inside a tile, one row, all three tile widths, and the width beside it that has a LayerNorm launch.
Metric: max|gpu - oracle| / max|oracle| <= 2e-2 (bf16 storage)."""
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seq,samples", [(1, 1), (33, 1), (77, 1), (77, 3)])
@pytest.mark.parametrize("heads", [4, 6, 8, 12, 16])
def test_layer_norm_inside_the_projections(heads, seq, samples):
    import torch
    from oracle import text_encoder
    from paper_2405_01248_amd.harness import DeviceEncoder, rel_err
    cfg = si.EncoderConfig(f"norm_{heads}_{seq}_{samples}", "bf16", 2, 64 * heads, heads, 64, seq, 512, 256 * heads, samples)
    inp = si.make_encoder_inputs(cfg, seed=heads + seq)
    de = DeviceEncoder(cfg, inp)
    ref = text_encoder.encoder_fwd(inp["params"], inp["ids"], cfg.n_layers, cfg.n_heads, cfg.ln_eps)
    de.run_slices(samples)
    torch.cuda.synchronize()
    assert rel_err(de.output(), ref) <= 2e-2
    # the embedding alone, and the layers from it on: the state between calls is in the storage dtype
    le = cfg.n_layers + 2
    de.hidden.zero_()
    for lo, hi in ((0, 1), (1, 2), (2, le)):
        de.enc.fwd_partial(de.params, de.ids, de.hidden, de.gb, lo, hi, 0, samples, de.ws)
    torch.cuda.synchronize()
    assert rel_err(de.output(), ref) <= 2e-2
