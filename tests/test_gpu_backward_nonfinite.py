"""A token that no expert kept has no part in any gradient, whatever its rows of dout and x hold (a masked token of a step whose
loss overflowed).  Contractions over an expert's rows are padded; experts without rows, of a row or two, at and around the
padded lengths, and both sides of the expected row count and of the capacities that decide how the rows are read.  The
gradients equal, bit for bit, those with finite rows, and those the oracle's."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu

# (dtype, T, d, H, C, rows of each expert); two experts to a token: T / 3 rows expected of each of the six
CASES = [
    (I.DT_BF16, 384, 136, 96, 190, (0, 1, 63, 64, 128, 190)),       # 128 expected: copies
    (I.DT_BF16, 387, 136, 96, 190, (0, 1, 63, 64, 128, 190)),       # 129, a padded capacity of 192: copies
    (I.DT_BF16, 387, 136, 96, 250, (0, 1, 64, 191, 192, 250)),      # 129, a padded capacity of 256: rows of x fetched
    (I.DT_BF16, 700, 264, 200, 330, (0, 2, 255, 256, 257, 330)),    # fetched, a product for each gate; a ragged last column tile
    (I.DT_BF16, 700, 264, 264, 8192, (0, 1, 255, 256, 257, 690)),   # dout fetched as well
    (I.DT_BF16, 300, 136, 200, 8200, (0, 1, 64, 65, 128, 290)),     # few rows of a large capacity, no multiple of 64
    (I.DT_BF16, 50000, 264, 96, 16900, (0, 1, 255, 256, 257, 16800)),         # 8192 or more expected: launches of their own
    (I.DT_BF16, 300, 64, 72, 200, (0, 1, 63, 64, 65, 200)),         # narrow: transposed copies
    (I.DT_F32, 300, 136, 72, 200, (0, 1, 31, 32, 33, 200)),
]


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype,T,d,Hh,C,rows", CASES)
def test_dropped_token_leaves_no_trace(oracle, dtype, T, d, Hh, C, rows, bad):
    import gpu_helpers as H
    B.load_library()
    E = len(rows)
    shape = I.EtrShape("nonfinite", 37, T=T, d=d, E=E, D=8, k=2, capacity=C, H=Hh, dtype=dtype, mode=I.MODE_BIDIR, recipe="iso",
                       n_centroids=E)
    print(f"dropped token dtype={dtype} T={T} d={d} H={Hh} C={C} bad={bad}", flush=True)
    L = H.GpuLayer(shape)
    L.route()
    slot_of, slot_token = np.full((T, E), -1, np.int32), np.full((E, C), -1, np.int32)
    rng = np.random.default_rng(3)
    for e, n in enumerate(rows):                         # any tokens but the first, ascending
        tokens = np.sort(rng.choice(np.arange(1, T), n, replace=False))
        slot_token[e, :n] = tokens
        slot_of[tokens, e] = np.arange(n)
    tables = [torch.from_numpy(v).cuda() for v in (slot_of, slot_token, np.array(rows, np.int32))]
    dout = I.make_upstream_gradient(shape, "cuda")
    dout[0] = 0
    ws = B.alloc_workspace(B.etr_backward_workspace_bytes(L.cfg))

    def backward(x, dout):
        out = [torch.full(s, 7.0, dtype=shape.torch_dtype, device="cuda") for s in ((T, d), (E, Hh, d), (E, Hh, d), (E, d, Hh))]
        ws.fill_(0xFF)
        B.etr_moe_backward(L.cfg, x, *(L.t[n] for n in ("w_emb", "w_gate", "w_up", "w_down")), L.score, L.gate, *tables, dout, *out, ws)
        torch.cuda.synchronize()
        return out

    names = ("dx", "dw_gate", "dw_up", "dw_down")
    want = backward(L.t["x"], dout)
    hx = L.host_inputs()
    ref = oracle.moe_backward(*(hx[n] for n in ("x", "w_emb", "w_gate", "w_up", "w_down")), slot_of, H.to_np(dout), D=8, dtype=dtype)
    for name, v in zip(names, want):
        a = oracle.to_f64(H.to_np(v), dtype)
        assert H.scale_rel_err(a, ref[name]) <= H.TOL_OUT[dtype], name
        if name != "dx":
            assert not a[0].any(), name                  # no rows: exact zeros
    dout[0] = bad
    for name, v, w in zip(names, backward(L.t["x"], dout), want):
        assert torch.equal(v, w), name
    x = L.t["x"].clone()
    x[0] = bad                                           # (its own input gradient is then what it may be)
    for name, v, w in zip(names, backward(x, dout), want):
        assert torch.equal(v[1:] if name == "dx" else v, w[1:] if name == "dx" else w), name
