"""Workspace sizes, on the host: a workspace sized for a number of samples serves every call of fewer."""
import pytest

from paper_2405_01248_amd import binding as B


@pytest.mark.parametrize("width", [128, 256, 640, 768, 1024, 2048])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_text_encoder_workspace_grows_with_the_samples(width, mode):
    enc = B.Encoder(B.DP_BF16, 2, width, width // 64, 64, 77, 1000, 4 * width)
    enc.set_batch_invariant(mode)
    sizes = [enc.workspace_bytes(n) for n in list(range(1, 129)) + [200, 500, 1000]]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_image_encoder_workspace_grows_with_the_samples():
    from synth_inputs import vae_encoder_layers
    layers = vae_encoder_layers(32, (1, 2, 4, 4), 8, 8)
    for h, w in ((64, 64), (384, 328), (512, 512)):
        enc = B.ImageEncoder(B.DP_BF16, h, w, 8, 32, layers)
        for lo, hi in ((0, len(layers)), (len(layers) - 3, len(layers))):
            sizes = [enc.workspace_bytes(lo, hi, n) for n in range(1, 40)]
            assert all(a <= b for a, b in zip(sizes, sizes[1:]))


@pytest.mark.parametrize("kind", [B.KIND_UNET, B.KIND_DIT])
def test_short_stages_hold_one_set_of_backward_buffers(kind):
    # a second set is for stages that use the side stream; two blocks on one stream share theirs, but for what one hands to the next
    t, d = 8 * 1024, 640
    size = lambda blocks: B.Stage(kind, B.DP_BF16, blocks, 8, 1024, d, 10, 64, 77, 768, 4 * d).workspace_bytes(True)
    second, later = size(2) - size(1), size(5) - size(4)
    assert second - later <= t * d * 2 + (1 << 20) + (0 if kind == B.KIND_UNET else 16 * t * d // 2)
    assert size(3) - size(2) > later + 4 * t * d * 2


def test_attention_buffers_of_the_image_encoder_take_no_room_beside_the_large_layers():
    from synth_inputs import vae_encoder_layers
    layers = vae_encoder_layers(128, (1, 2, 4, 4), 8, 8)
    size = lambda l, n: B.ImageEncoder(B.DP_BF16, 512, 512, 8, 32, l).workspace_bytes(0, len(l), n)
    without = tuple(x for x in layers if x[0] != "attn")
    for n in (1, 4, 8):
        assert size(layers, n) <= size(without, n) + (1 << 20)
