"""The backward's products whose operands lie with the contraction index slow, at the edges of their kernel's tiles: the
fewest k-tiles, halves of a split contraction that end inside a k-tile, outputs narrower than one tile and ragged ones, more
tiles than workgroups with few k-tiles each, and contraction rows fetched through an index over short, empty and long
experts.  Against the oracle with the layer's tolerance, and a second call on the used workspace gives the same bits."""
import pytest

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


# (T, E, d, H, C, k, recipe).  The contraction of u is d, that of the input gradient H and H, that of the weight gradients the
# kept rows (at least 128; 256 where rows are fetched through the slot list: of x with more than 128 rows expected, of x and dout
# from a capacity of 8192 on).
CASES = [
    (300, 4, 128, 64, 128, 1, "bias"),          # two k-tiles everywhere; outputs of 64 and 128 columns
    (300, 4, 136, 72, 100, 2, "bias"),          # halves of 72: a whole and a short k-tile each
    (300, 2, 128, 120, 300, 2, "iso"),          # halves of 120
    (700, 3, 200, 264, 400, 2, "bias"),         # one column past a tile of 256, contraction of 200
    (2000, 16, 128, 2056, 200, 2, "cluster"),   # many short tiles per workgroup
    (1500, 8, 1160, 520, 700, 3, "zipf"),       # ragged both ways, uneven experts
    (900, 4, 264, 72, 8192, 2, "bias"),         # fetched rows, capacity above the tokens
    (2000, 16, 128, 264, 20000, 2, "bias"),     # a list of tiles whose live ones lie far apart
    (9000, 6, 136, 136, 8200, 2, "zipf"),       # fetched rows, capacity no multiple of 64, experts from few rows to thousands
]


@pytest.mark.parametrize("T,E,d,Hh,C,k,recipe", CASES)
def test_transposed_products(oracle, T, E, d, Hh, C, k, recipe):
    import gpu_helpers as H
    from test_gpu_backward import Backward, _err
    B.load_library()
    shape = I.EtrShape("transposed", 17, T=T, d=d, E=E, D=8, k=k, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_BIDIR,
                       recipe=recipe, n_centroids=E)
    print(f"transposed products T={T} E={E} d={d} H={Hh} C={C}", flush=True)
    bw = Backward(H, shape, shape.mode)                  # (its workspace is filled with NaN patterns)
    hb = bw.host()
    ref = oracle.moe_backward(hb["x"], hb["w_emb"], hb["w_gate"], hb["w_up"], hb["w_down"], hb["slot_of"], hb["dout"],
                              D=shape.D, dtype=shape.dtype)
    names = (("dx", "dx"), ("dwg", "dw_gate"), ("dwu", "dw_up"), ("dwd", "dw_down"))
    for got, key in names:
        assert _err(H, oracle, getattr(bw, got), ref[key], shape.dtype) <= H.TOL_OUT[shape.dtype], key
    bw.check_second_call()
