"""Pooling groups of whole 16-byte pieces whose number is no power of two (3, 5, 7, 9 pieces: one, two and three passes of
four requests), more and fewer groups than lanes, more experts than one staging pass takes."""
import pytest

from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,D,dtype,cos", [(130, 1080, 12, 24, I.DT_BF16, I.COS_POOLED), (5000, 2496, 33, 24, I.DT_BF16, I.COS_FULL),
                                               (70, 400, 7, 40, I.DT_BF16, I.COS_FULL), (33, 560, 64, 8, I.DT_F32, I.COS_FULL),
                                               (65, 112, 2, 56, I.DT_BF16, I.COS_POOLED), (40, 720, 16, 36, I.DT_F32, I.COS_FULL),
                                               (3, 1200, 50, 12, I.DT_F32, I.COS_POOLED)])
def test_route_groups(oracle, T, d, E, D, dtype, cos):
    import gpu_helpers as H
    import test_gpu_parity
    from paper_2406_00023_amd import binding as B
    B.load_library()
    test_gpu_parity.test_route(H, oracle, T, d, E, D, dtype, cos)
