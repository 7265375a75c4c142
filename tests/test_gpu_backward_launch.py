"""The backward's last products in one launch, where their division can go wrong.  bf16 with few rows: the input gradient's
contraction in parts (the last one shorter, one that begins in the first half and ends in the second, halves that end inside a
k-tile, more than one row tile, a narrow last column tile).  fp32: both tile sizes, widths that end inside a tile, halves that
end inside a k-step, empty experts and experts of a row or two, a capacity above the rows.  Against the oracle with the layer's
tolerance, and a second call on the used workspace gives the same bits."""
import pytest

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu

# (dtype, T, E, d, H, C, k, recipe); parts of the contraction (k-tiles of each) on 256 CUs
CASES = [
    (I.DT_BF16, 300, 2, 136, 1000, 100, 2, "bias"),      # 11 + 11 + 10 of twice 16, the halves ending inside a k-tile
    (I.DT_BF16, 40, 3, 128, 840, 64, 1, "iso"),          # 14 + 14, each a half
    (I.DT_BF16, 64, 8, 1024, 2816, 64, 2, "cluster"),    # 30 + 30 + 28, four column tiles
    (I.DT_BF16, 500, 2, 520, 3000, 600, 2, "bias"),      # 7 parts; three row tiles of the capacity, fetched rows of x
    (I.DT_BF16, 100, 2, 128, 5000, 128, 1, "zipf"),      # 8 parts
    (I.DT_BF16, 1000, 2, 128, 4000, 900, 2, "zipf"),     # 8 parts wanted, 6 that the workspace holds
    (I.DT_F32, 37, 2, 24, 40, 40, 1, "bias"),            # everything inside one tile
    (I.DT_F32, 5, 8, 64, 200, 64, 1, "cluster"),         # empty experts, one or two rows
    (I.DT_F32, 300, 4, 136, 72, 100, 2, "bias"),         # 32 x 32 tiles, ragged
    (I.DT_F32, 700, 12, 520, 264, 600, 3, "zipf"),       # 64 x 64 tiles, ragged, uneven experts
    (I.DT_F32, 400, 16, 256, 1000, 4000, 1, "zipf"),     # capacity above the tokens
]


@pytest.mark.parametrize("dtype,T,E,d,Hh,C,k,recipe", CASES)
def test_products_in_one_launch(oracle, dtype, T, E, d, Hh, C, k, recipe):
    import gpu_helpers as H
    from test_gpu_backward import Backward, _err
    B.load_library()
    shape = I.EtrShape("one_launch", 23, T=T, d=d, E=E, D=8, k=k, capacity=C, H=Hh, dtype=dtype, mode=I.MODE_BIDIR,
                       recipe=recipe, n_centroids=E)
    print(f"backward launch dtype={dtype} T={T} E={E} d={d} H={Hh} C={C}", flush=True)
    bw = Backward(H, shape, shape.mode)                  # (its workspace is filled with NaN patterns)
    hb = bw.host()
    ref = oracle.moe_backward(hb["x"], hb["w_emb"], hb["w_gate"], hb["w_up"], hb["w_down"], hb["slot_of"], hb["dout"],
                              D=shape.D, dtype=shape.dtype)
    names = (("dx", "dx"), ("dwg", "dw_gate"), ("dwu", "dw_up"), ("dwd", "dw_down"))
    for got, key in names:
        assert _err(H, oracle, getattr(bw, got), ref[key], shape.dtype) <= H.TOL_OUT[shape.dtype], key
    bw.check_second_call()
