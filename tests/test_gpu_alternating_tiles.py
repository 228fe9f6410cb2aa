"""GPU parity of the GEMM tiles whose waves work in two alternating groups (y = x W^T, and the grouped dW = dy^T x) at the
sizes where they can go wrong: one tile and less, ragged edges on both sides, a contraction of one k-tile, of a number of
k-tiles that is odd or below the pipeline's depth, and of a part of a k-tile at its end."""
import pytest

from test_gpu_ops import TOL_BF16, TOL_F32OUT, _gemm_case

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 8), (256, 256, 64), (77, 264, 128), (300, 520, 192), (257, 136, 72), (512, 200, 320), (333, 392, 1000)]


@pytest.mark.parametrize("tile_cfg", [18, 19, 20, 21])
def test_forward_tiles(tile_cfg):
    for M, N, K in SHAPES:
        e = _gemm_case("nt", M, N, K, tile_cfg, seed=M + K)
        print(f"\n[gemm nt cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_BF16


@pytest.mark.parametrize("K", [64, 128, 320])
@pytest.mark.parametrize("tile_cfg,width", [(18, 256), (19, 128), (20, 192), (21, 160)])
def test_workgroups_that_walk_over_tiles(tile_cfg, width, K):
    # beyond 256 tiles: two of 256 workgroups take a second tile; all but two take a second one, ragged on both sides; 1, 2 and 5 k-tiles
    for M, N in [(43 * 256, 6 * width), (34 * 256 - 3, 15 * width - 8)]:
        e = _gemm_case("nt", M, N, K, tile_cfg, seed=M + K)
        print(f"\n[gemm nt cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_BF16


@pytest.mark.parametrize("K", [64, 320, 1088])
@pytest.mark.parametrize("tile_cfg,width", [(18, 256), (20, 192)])
def test_one_round_of_tiles_on_either_instruction(tile_cfg, width, K):
    # from 160 tiles on the 16x16x32 instruction, transposed on its way to the epilogue, 256 columns only where few CUs idle through few k-tiles (200 tiles: not through
    # the 17 of the longest); below it the 32x32x16 one; ragged on both sides
    for M, N in [(40 * 256 - 5, 4 * width + 16), (39 * 256 + 3, 3 * width + 8), (39 * 256, 3 * width + 200)]:
        e = _gemm_case("nt", M, N, K, tile_cfg, seed=M + K)
        print(f"\n[gemm nt cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_BF16


@pytest.mark.parametrize("kind", ["dit", "unet"])
def test_stage_of_more_tiles_than_compute_units(kind):
    # the kinds of epilogue of a stage behind workgroups that walk over tiles: 259 row tiles, the last one ragged
    import torch
    import synth_inputs as si
    from paper_2405_01248_amd.harness import DeviceStage
    from test_gpu_parity import _compare, _oracle_stage
    ctx = (0, 0) if kind == "dit" else (8, 64)
    cfg = si.StageConfig("walk_" + kind, si.DIT if kind == "dit" else si.UNET, "bf16", 1, 331, 200, 128, 2, 64, *ctx, 512, 1e-6 if kind == "dit" else 1e-5, int(kind == "dit"))
    inp = si.make_stage_inputs(cfg, seed=3)
    ds = DeviceStage(cfg, inp)
    ds.step()
    torch.cuda.synchronize()
    _compare(cfg, ds.results(), _oracle_stage(cfg, inp))


@pytest.mark.parametrize("layout", ["nt", "nn"])
@pytest.mark.parametrize("tile_cfg", [26, 27, 28, 29])
def test_tiles_whose_waves_share_the_contraction(tile_cfg, layout):
    # fewer k-tiles than waves, as many, one more; a part of a tile and ragged edges; weights [out, in] and as a product dx = dy W finds them
    for M, N, K in [(8, 8, 64), (64, 96, 256), (77, 264, 320), (129, 136, 192), (300, 520, 1088)]:
        e = _gemm_case(layout, M, N, K, tile_cfg, seed=M + K)
        print(f"\n[gemm {layout} cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_BF16


@pytest.mark.parametrize("layout", ["nt", "nn"])
@pytest.mark.parametrize("tile_cfg,width", [(30, 32), (31, 64), (32, 96)])
def test_32_rows_with_eight_waves_that_share_the_contraction(tile_cfg, width, layout):
    # fewer k-tiles than waves, as many, one more, two rounds; one row more and less than a tile, a ragged column edge, one CU with two tiles
    for M, N, K in [(8, 8, 64), (32, width, 512), (33, width + 8, 576), (77, 3 * width - 8, 1024), (65, 264 * width // 2, 320), (31, 520, 1088)]:
        e = _gemm_case(layout, M, N, K, tile_cfg, seed=M + K)
        print(f"\n[gemm {layout} cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_BF16


@pytest.mark.parametrize("M,N,K", [(4064, 112, 512), (4128, 112, 512), (8160, 104, 2048), (8200, 104, 2048)])
def test_few_columns_on_either_side_of_512_tiles_of_32_rows(M, N, K):
    # 508 and 516 tiles of 32x32, 510 and 514 of 32x64: beyond 512 a tile of more rows is chosen
    e = _gemm_case("nt", M, N, K, 0, seed=M + K)
    assert e <= TOL_BF16, e


@pytest.mark.parametrize("K", [64, 256, 320, 512, 576, 832, 1088])
def test_waves_with_one_and_two_k_tiles_on_their_way(K):
    # up to 256 tiles of 64x64 a wave has two k-tiles on their way to LDS, beyond one: 1, 2, 3, 4, 5 k-tiles of the first wave, fewer of the others
    for M, N in [(70, 136), (1100, 1048)]:
        e = max(_gemm_case(layout, M, N, K, 26, seed=M + K) for layout in ("nt", "nn"))
        print(f"\n[gemm nt cfg 26 {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_BF16


@pytest.mark.parametrize("tile_cfg", [22, 23, 24, 25])
@pytest.mark.parametrize("accumulate", [False, True])
def test_weight_gradient_tiles(tile_cfg, accumulate):
    for M, N, K in [(8, 8, 8), (256, 256, 64), (328, 392, 1000), (264, 136, 72), (64, 520, 2053)]:
        e = _gemm_case("tn", M, N, K, tile_cfg, seed=M + K, bias=False, accumulate=accumulate)
        print(f"\n[gemm tn cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_F32OUT


@pytest.mark.parametrize("tile_cfg", [22, 23, 24, 25])
@pytest.mark.parametrize("K", [64, 66, 128, 130, 192, 255, 320, 1025])
def test_weight_gradient_with_k_tiles_turned_round(tile_cfg, K):
    # 3 x 3 tiles or more, every other one with its k-tiles in pairs turned round: one to five k-tiles, whole and ragged at either end of a pair, and parts
    for M, N in [(520, 776), (776, 520)]:
        e = _gemm_case("tn", M, N, K, tile_cfg, seed=M + K, bias=False, accumulate=False)
        assert e <= TOL_F32OUT, (M, N, K, e)


@pytest.mark.parametrize("M,N,K", [(4090, 4088, 256), (4100, 4616, 128), (2060, 1544, 384)])
def test_fp8_tiles(M, N, K):
    # 256, 192 and 128 columns wide, ragged on both sides
    import test_gpu_ops
    test_gpu_ops.test_fp8_gemm_matches_oracle(M, N, K)


@pytest.mark.parametrize("batch", [1, 16, 17, 40, 49])
def test_dit_stage_by_batch_size(batch):
    # the modulation projections: 1, 2, 3 row tiles of the few-rows kernel, one launch for all blocks, and the tile kernels beyond
    import numpy as np
    import torch
    import synth_inputs as si
    from oracle import blocks
    from paper_2405_01248_amd.harness import DeviceStage, rel_err
    cfg = si.StageConfig("dit_batch", si.DIT, "bf16", 2, batch, 8, 160, 2, 80, 0, 0, 320, 1e-6, 1)
    inp = si.make_stage_inputs(cfg, seed=batch)
    ds = DeviceStage(cfg, inp)
    ds.step()
    torch.cuda.synchronize()
    got = ds.results()
    y, caches = blocks.stage_fwd(cfg.kind, inp["params"], inp["x"], inp["cond"], cfg.n_blocks, cfg.n_heads, cfg.ln_eps, gelu_tanh=True)
    e = rel_err(got["y"], y)
    assert np.isfinite(got["y"]).all() and e <= TOL_BF16, e


@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (32, 32, 16), (33, 36, 20), (65, 68, 132), (40, 96, 260)])
@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_f32_gemm(layout, M, N, K):
    import numpy as np
    import torch
    from paper_2405_01248_amd import binding as B
    a_k, b_k = {"nt": (0, 0), "nn": (0, 1), "tn": (1, 1)}[layout]
    rng = np.random.default_rng(M + K)
    A, Bm = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    dA = torch.from_numpy(np.ascontiguousarray(A.T if a_k else A)).cuda()
    dB = torch.from_numpy(np.ascontiguousarray(Bm if b_k else Bm.T)).cuda()
    out = torch.zeros((M, N), device="cuda")
    B.op_gemm(B.DP_F32, dA, dA.shape[1], a_k, dB, dB.shape[1], b_k, M, N, K, None, out, N, layout == "tn")
    torch.cuda.synchronize()
    ref = A.astype(np.float64) @ Bm.astype(np.float64)
    assert float(np.abs(out.cpu().numpy() - ref).max() / np.abs(ref).max()) <= 1e-5


@pytest.mark.parametrize("kind,batch,tokens,blocks", [("unet", 1, 128, 3), ("unet", 3, 43, 2), ("dit", 2, 64, 3), ("dit", 5, 26, 2)])
def test_f32_products_in_one_launch(kind, batch, tokens, blocks):
    # weight gradients over 128 rows (four waves) and over 129 and 130 (eight, ragged), of the context and the conditioning beside them; several
    # blocks, whose buffers lie in each other's place; widths that are no multiple of a tile
    import torch
    import synth_inputs as si
    from paper_2405_01248_amd.harness import DeviceStage
    from test_gpu_parity import _compare, _oracle_stage
    ctx = (7, 40) if kind == "unet" else (0, 0)
    cfg = si.StageConfig("f32_dw_" + kind, si.UNET if kind == "unet" else si.DIT, "f32", blocks, batch, tokens, 48, 2, 24, *ctx, 72, 1e-5 if kind == "unet" else 1e-6, int(kind == "dit"))
    inp = si.make_stage_inputs(cfg, seed=tokens)
    ds = DeviceStage(cfg, inp)
    ds.step()
    torch.cuda.synchronize()
    got = ds.results()
    _compare(cfg, got, _oracle_stage(cfg, inp))
    if kind == "unet":      # the GeGLU in the products around it changes no bit
        import numpy as np
        ds.stage.set_fusion(0)
        ds.step()
        torch.cuda.synchronize()
        plain = ds.results()
        assert np.array_equal(got["y"], plain["y"]) and np.array_equal(got["dx"], plain["dx"])
        assert all(np.array_equal(got["grads"][k], plain["grads"][k]) for k in plain["grads"])


@pytest.mark.parametrize("heads,d_head,batch,tokens,blocks", [(1, 64, 3, 9, 17), (9, 72, 33, 7, 2), (25, 80, 2, 5, 1)])
def test_dit_backward_by_width(heads, d_head, batch, tokens, blocks):
    # LayerNorm backward with the gated branch in it: one wave and four per row, ragged rows; the conditioning gradient: less than a column
    # tile, 33 rows, more blocks than one launch takes
    import numpy as np
    import torch
    import synth_inputs as si
    from oracle import blocks as ob
    from paper_2405_01248_amd.harness import DeviceStage, rel_err
    cfg = si.StageConfig("dit_width", si.DIT, "bf16", blocks, batch, tokens, heads * d_head, heads, d_head, 0, 0, 64, 1e-6, 1)
    inp = si.make_stage_inputs(cfg, seed=heads)
    ds = DeviceStage(cfg, inp)
    ds.step()
    torch.cuda.synchronize()
    got = ds.results()
    y, caches = ob.stage_fwd(cfg.kind, inp["params"], inp["x"], inp["cond"], cfg.n_blocks, cfg.n_heads, cfg.ln_eps, gelu_tanh=True)
    dx, dcond, grads = ob.stage_bwd(cfg.kind, inp["params"], caches, inp["dy"], cfg.n_heads)
    assert rel_err(got["y"], y) <= TOL_BF16
    assert rel_err(got["dx"], dx) <= TOL_BF16 and rel_err(got["dcond"], dcond) <= TOL_BF16
    for k in ("ada_w", "ada_b"):
        for b in range(blocks):
            name = [n for n in grads if n.startswith(f"block{b}.") and n.endswith(k)][0]
            assert rel_err(got["grads"][name], grads[name]) <= TOL_BF16, name


@pytest.mark.parametrize("batch,tokens,heads", [(2, 77, 8), (1, 77, 20), (2, 1024, 10), (4, 513, 4), (1, 513, 25)])
def test_geglu_fusion_changes_no_bit_of_the_forward(batch, tokens, heads):
    # sizes at which a plain projection takes tiles whose waves share the contraction, or 16x16 instructions: another order of additions; the
    # fused one 128x128, 256x256 and 256x128 tiles
    import numpy as np
    import torch
    import synth_inputs as si
    from paper_2405_01248_amd.harness import DeviceStage
    d = 64 * heads
    cfg = si.StageConfig("fusion_bits", si.UNET, "bf16", 1, batch, tokens, d, heads, 64, 7, 64, 4 * d)
    ds = DeviceStage(cfg, si.make_stage_inputs(cfg, seed=heads))
    y = []
    for mask in (3, 0):
        ds.stage.set_fusion(mask)
        ds.step()
        torch.cuda.synchronize()
        y.append(ds.results()["y"])
    assert np.array_equal(y[0], y[1])


@pytest.mark.parametrize("M,N,K,lda,ldb", [(5, 7, 1, 3, 5), (33, 34, 3, 0, 0), (65, 31, 130, 131, 133), (40, 41, 257, 0, 1), (64, 64, 64, 66, 0), (2097153, 4, 4, 0, 0)])
@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_f32_gemm_of_any_size_and_stride(layout, M, N, K, lda, ldb):
    # contractions and strides that are not multiples of 4; more row tiles than a grid's second dimension holds
    import torch
    from paper_2405_01248_amd import binding as B
    a_k, b_k = {"nt": (0, 0), "nn": (0, 1), "tn": (1, 1)}[layout]
    g = torch.Generator().manual_seed(M + K)
    A, Bm = torch.randn(M, K, generator=g), torch.randn(K, N, generator=g)
    stored = [A.T if a_k else A, Bm if b_k else Bm.T]
    dev = []
    for t, extra in zip(stored, (lda, ldb)):
        buf = torch.full((t.shape[0], t.shape[1] + extra), float("nan"))      # what lies between the rows is not read
        buf[:, :t.shape[1]] = t
        dev.append(buf.cuda())
    out = torch.zeros((M, N), device="cuda")
    B.op_gemm(B.DP_F32, dev[0], dev[0].shape[1], a_k, dev[1], dev[1].shape[1], b_k, M, N, K, None, out, N, layout == "tn")
    torch.cuda.synchronize()
    ref = A.double() @ Bm.double()
    assert float((out.cpu().double() - ref).abs().max() / ref.abs().max()) <= 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tokens", [4, 5])
def test_layer_norm_backward_with_an_infinite_gradient(dtype, tokens):
    """Weights that are zero but for one path carry the last row's gradient to the feed-forward's LayerNorm, where its first column overflows:
    that column's shift gradient is infinite, not NaN, and no other column's is touched, with an odd number of rows as with an even one."""
    import numpy as np
    import torch
    import synth_inputs as si
    from paper_2405_01248_amd.harness import DeviceStage
    cfg = si.StageConfig("overflow", si.UNET, dtype, 1, 1, tokens, 64, 1, 64, 3, 8, 64)
    inp = si.make_stage_inputs(cfg, seed=tokens)
    p = inp["params"]
    for k in ("ff_w1", "ff_b1", "ff_w2"):
        p["block0." + k] = np.zeros_like(p["block0." + k])
    p["block0.ff_w2"][0, 0] = 1.0
    p["block0.ff_b1"][64] = 8.0                # gate of the first hidden column: gelu(8) = 8, gelu'(8) = 1
    p["block0.ff_w1"][0, 0] = 4.0
    inp["dy"][0, -1, 0] = 2.0 ** 124           # times 8, times 4: 2^129
    ds = DeviceStage(cfg, inp)
    ds.step()
    torch.cuda.synchronize()
    g = ds.results()["grads"]["block0.ln3_b"]
    assert g[0] == np.inf and np.isfinite(g[1:]).all(), g[:4]


@pytest.mark.parametrize("batch,heads,d_head,cut", [(32, 12, 64, False), (48, 6, 64, True)])
def test_weight_gradients_are_cut_where_that_is_faster(batch, heads, d_head, cut):
    # 8192 rows of 768: tiles of 256x128 in whole rounds 120 us, 256x256 ones in two parts 126; 12288 rows of 384 fill the chip only in parts
    import torch
    import synth_inputs as si
    from paper_2405_01248_amd import binding as B
    from paper_2405_01248_amd.harness import DeviceStage
    d = heads * d_head
    cfg = si.StageConfig(f"dw_plan_{d}", si.DIT, "bf16", 1, batch, 256, d, heads, d_head, 0, 0, 4 * d, 1e-6, 1)
    ds = DeviceStage(cfg, si.make_stage_inputs(cfg, seed=0))
    ds.step()
    B.ktime_begin(256)
    ds.step()
    launches = [(r["kind"], r["m"], r["n"]) for r in B.ktime_end(256)]
    torch.cuda.synchronize()
    assert sum(k == "gemm_tn" for k, _, _ in launches) == 1
    assert (("reduce", d, 4 * d) in launches) == cut, launches
