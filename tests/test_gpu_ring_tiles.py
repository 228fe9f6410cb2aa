"""GPU parity of the 64x64 and 128x128 rings of direct-to-LDS buffers: contractions of fewer k-tiles than buffers, as many and more, on few tiles (four
buffers) and, for 64x64, on more than 512 (three)."""
import pytest

from test_gpu_ops import TOL_BF16, _gemm_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_cfg,M,N", [(16, 77, 136), (16, 1530, 1480), (14, 77, 136), (14, 300, 264)])
def test_ring_of_buffers(tile_cfg, M, N):
    for K in (64, 128, 192, 256, 320, 384, 448, 576):
        e = _gemm_case("nt", M, N, K, tile_cfg, seed=M + K)
        assert e <= TOL_BF16, (K, e)


@pytest.mark.parametrize("heads", [8, 12, 16])
def test_segments_in_a_workgroup_and_parts_of_a_launch_agree(heads):
    """Batch-invariant mode 1 on 1 sample (parts of their own), 5, 13 and 25 (the parts one after the other in a workgroup, 64x64 tiles and larger ones): the same bits."""
    import numpy as np
    import torch
    import synth_inputs as si
    from paper_2405_01248_amd.harness import DeviceEncoder
    cfg = si.EncoderConfig(f"segments_{heads}", "bf16", 2, 64 * heads, heads, 64, 77, 512, 256 * heads, 25)
    de = DeviceEncoder(cfg, si.make_encoder_inputs(cfg, seed=heads))
    de.enc.set_batch_invariant(1)
    de.ws = torch.empty(de.enc.workspace_bytes(de.gb), dtype=torch.uint8, device=de.device)
    outs = []
    for sizes in ((25,), (13, 12), (5,) * 5, (1,) * 25):
        de.hidden.zero_()
        off = 0
        for n in sizes:
            de.enc.fwd_partial(de.params, de.ids, de.hidden, de.gb, 0, cfg.n_layers + 2, off, n, de.ws)
            off += n
        torch.cuda.synchronize()
        outs.append(de.output())
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])


@pytest.mark.parametrize("M,N,K", [(616, 1280, 768), (616, 2304, 768), (308, 3072, 768), (616, 3072, 768), (1232, 1280, 1024)])
def test_products_of_a_few_hundred_rows_keep_their_order_of_additions(M, N, K):
    """The context projection of a U-Net block and a text encoder's projections on 4 to 16 samples: partial sums of four waves, whatever the 64x64 ring takes for
    them.  (The ring adds the k-tiles up in one sum.)"""
    import torch
    from paper_2405_01248_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    a = torch.randn((M, K), generator=gen, device="cuda").bfloat16()
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.05).bfloat16()
    out = []
    for tile_cfg in (0, 26, 16):
        c = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        B.op_gemm(B.DP_BF16, a, K, 0, w, K, 0, M, N, K, None, c, N, False, False, None, tile_cfg)
        out.append(c)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1]) and not torch.equal(out[0], out[2])
