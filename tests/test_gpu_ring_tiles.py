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
