"""Text-encoder calls of few rows, whose projections normalise their rows themselves (widths of 256 to 1024 that are multiples of 256, 32-row tiles, one a CU at
most), against the fp64 oracle: rows that end inside a tile, one row, and the width beside it that has a LayerNorm launch.
Metric: max|gpu - oracle| / max|oracle| <= 2e-2 (bf16 storage).  And, with weights that hand the normalised rows through, the bits of a LayerNorm launch; the recorded launches
show which of the two ran."""
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


def _one_row_samples(heads, rows, through_fc1, eps=1e-37):
    """An encoder of one layer on samples of one row, whose output shows the bits of a LayerNorm of `rows` rows: a projection of ones and zeros takes its result to the
    residual (the values, attention over one key, an out-projection of ones and zeros; or both halves of the feed-forward), which is 2^-30 of it.  Half of a
    row's values are one number and half another, so that the result is +-1; a shift of -1 leaves of the former what mean and deviation
    round to."""
    import numpy as np
    from paper_2405_01248_amd.harness import DeviceEncoder
    d = 64 * heads
    cfg = si.EncoderConfig(f"rows_{d}_{rows}", "bf16", 1, d, heads, 64, 1, rows, 4 * d, rows, 1, eps)
    inp = si.make_encoder_inputs(cfg, seed=heads)
    rng = np.random.default_rng(heads)
    p = inp["params"]
    for name in p:
        p[name] = np.zeros(p[name].shape)
    ranks = np.argsort(rng.random((rows, d)), axis=1) % 2
    p["tok_emb"] = si.round_bf16(2.0 ** -30 * (rng.uniform(-4, 4, (rows, 1)) + rng.uniform(0.5, 2, (rows, 1)) * (2 * ranks - 1)))
    eye = np.eye(d)
    for n in ("ln1", "ln2"):
        p[f"layer0.{n}_g"] = np.ones(d)
        p[f"layer0.{n}_b"] = -np.ones(d)
    if through_fc1:
        p["layer0.fc1_w"][:d] = eye
        p["layer0.fc2_w"][:, :d] = eye
    else:
        p["layer0.wqkv"][2 * d:] = eye
        p["layer0.wo"] = eye
    inp["ids"] = np.arange(rows).reshape(rows, 1)
    return DeviceEncoder(cfg, inp)


def _layers(de, rows):
    """Embedding and layer on slices of that many rows, and the recorded launches of the first slice."""
    import torch
    from paper_2405_01248_amd import binding as B
    de.hidden.zero_()
    B.ktime_begin(64)
    de.enc.fwd_partial(de.params, de.ids, de.hidden, de.gb, 0, 2, 0, rows, de.ws)
    launches = B.ktime_end(64)
    de.run_slices(rows, 0, 2)
    torch.cuda.synchronize()
    return de.hidden.clone(), launches


def _normalises(launches, n, k):
    """Whether the projection to n columns read its rows in fp32."""
    r, = [r for r in launches if r["kind"] == "gemm_nt" and (r["n"], r["k"]) == (n, k)]
    return r["bytes"] >= 2 * (2 * r["m"] * k + n * k + r["m"] * n)


@pytest.mark.parametrize("through_fc1", [False, True])
@pytest.mark.parametrize("heads", [4, 8, 12, 16])
def test_rows_normalised_inside_the_product_have_the_bits_of_a_launch(heads, through_fc1):
    # 308 rows of width 768 before the first projection: 96-column tiles, beside the narrower ones of the others
    import torch
    d = 64 * heads
    n = 4 * d if through_fc1 else 3 * d
    de = _one_row_samples(heads, 2048, through_fc1)
    launched, launches = _layers(de, 2048)
    assert sum(r["kind"] == "ln_fwd" for r in launches) == 2 and not _normalises(launches, n, d)
    for rows in (1, 33, 77, 308):
        inside, launches = _layers(de, rows)
        assert _normalises(launches, n, d) or rows == 308 and (heads, through_fc1) != (12, False), rows
        assert torch.equal(inside.view(torch.int16), launched.view(torch.int16)), rows


@pytest.mark.parametrize("through_fc1", [False, True])
def test_infinities_and_nan_stay_in_their_rows(through_fc1):
    import torch
    de = _one_row_samples(12, 2048, through_fc1)
    emb = de.params[0]
    emb[5, 300], emb[40, 0], emb[77, 767] = float("inf"), float("nan"), float("-inf")
    launched, _ = _layers(de, 2048)
    inside, launches = _layers(de, 77)
    assert _normalises(launches, (4 if through_fc1 else 3) * 768, 768)
    bad = launched[:, 0].isnan().all(dim=1)
    assert bad.nonzero().flatten().tolist() == [5, 40, 77]
    assert torch.equal(inside[bad].isnan(), launched[bad].isnan()) and torch.equal(inside[~bad], launched[~bad])
