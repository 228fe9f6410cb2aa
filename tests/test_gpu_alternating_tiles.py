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


@pytest.mark.parametrize("tile_cfg", [22, 23, 24, 25])
@pytest.mark.parametrize("accumulate", [False, True])
def test_weight_gradient_tiles(tile_cfg, accumulate):
    for M, N, K in [(8, 8, 8), (256, 256, 64), (328, 392, 1000), (264, 136, 72), (64, 520, 2053)]:
        e = _gemm_case("tn", M, N, K, tile_cfg, seed=M + K, bias=False, accumulate=accumulate)
        print(f"\n[gemm tn cfg {tile_cfg} {M}x{N}x{K}] rel err {e:.2e}", flush=True)
        assert e <= TOL_F32OUT


@pytest.mark.parametrize("M,N,K", [(4090, 4088, 256), (4100, 4616, 128), (2060, 1544, 384)])
def test_fp8_tiles(M, N, K):
    # 256, 192 and 128 columns wide, ragged on both sides
    import test_gpu_ops
    test_gpu_ops.test_fp8_gemm_matches_oracle(M, N, K)
