"""The order in which the persistent kernel walks its tiles: groups of 5 to 8 row tiles, which lie in one super-tile whole, with
column tiles that fill the last super-tile or not, and experts from no rows to all of their capacity, against the oracle."""
import pytest

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


# (capacity, d, H, rows of each expert): 5 x 6, 6 x 5, 7 x 4 and 8 x 4 tiles; ragged column tiles and contractions too
@pytest.mark.parametrize("C,d,Hh,rows", [
    (1280, 256, 1664, (1280, 0, 1025, 300, 1)), (1500, 512, 896, (1281, 1500, 7, 1024, 0, 512)),
    (1600, 264, 520, (1600, 1537, 256, 1000)), (2048, 256, 1152, (2048, 1793, 900, 2000)), (1900, 328, 1096, (5, 1900, 1600, 1792))])
def test_groups_of_five_to_eight_row_tiles(oracle, C, d, Hh, rows):
    import gpu_helpers as H
    B.load_library()
    E = len(rows)
    shape = I.EtrShape("super_tiles", 41, T=E * C, d=d, E=E, D=8, k=1, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_BIDIR, recipe="iso")
    print(f"super-tiles C={C} d={d} H={Hh} rows={rows}", flush=True)
    assert H.ffn_plan(B.make_config(shape), 0, gathered=False)[0] in (H.PERSISTENT, H.PERSISTENT_TAIL)
    H.check_expert_ffn(oracle, shape, list(rows))
