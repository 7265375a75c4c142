"""The fp32 grouped GEMM at the edges of its tiles: both tile sizes (64 x 64 from two tiles per CU on, else 32 x 32), row
counts on and next to tile boundaries, empty experts, contractions that end inside a k-tile of 32."""
import pytest

from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,C,d,Hh,counts", [
    (8, 520, 264, 520, [520, 0, 1, 64, 65, 128, 513, 63]),      # gate/up on 64 x 64, down on 32 x 32, short last k-tiles
    (3, 100, 40, 72, [100, 33, 32]),                            # 32 x 32, two k-tiles (the second short)
    (2, 31, 8, 8, [31, 1]),                                     # one short k-tile, narrower than a tile
    (64, 64, 128, 512, [64, 0, 7, 33] * 16),                    # as many experts as a wave has lanes
    (1, 2100, 1032, 1096, [2100]),                              # 64 x 64 in both products
])
def test_f32_gemm_edges(oracle, E, C, d, Hh, counts):
    import gpu_helpers as H
    import test_gpu_parity
    from paper_2406_00023_amd import binding as B
    B.load_library()
    test_gpu_parity.test_expert_ffn(H, oracle, I.DT_F32, E, C, d, Hh, counts)
