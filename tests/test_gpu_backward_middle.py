"""The element-wise middle of the bf16 backward, a pass of its own where few tiles are expected and else the epilogue of its product,
here also behind the second and third tile of a workgroup: experts whose rows end inside the pieces of 8 and
the blocks of 32 rows that it goes by, in the second half of a tile, past one tile, and none at all; widths that end inside a
piece of 64 hidden units; kept pre-activations and recomputed ones, -1 in the slot list behind an expert's rows.  All gradients, with that
of the gate, against the oracle with the layer's tolerance; the workspace holds NaN patterns."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


# (T, d, H, C, rows of each expert)
@pytest.mark.parametrize("T,d,Hh,C,rows", [
    (120, 128, 72, 100, (1, 7, 8, 9, 31, 32, 33, 100)), (400, 136, 64, 300, (0, 127, 128, 129, 255, 256, 257, 300)),
    (700, 264, 328, 640, (159, 160, 161, 512, 513, 640, 2, 64)), (200, 128, 1024, 200, (65, 0, 200)),
    (900, 128, 200, 8192, (0, 1, 255, 256, 257, 900))])
@pytest.mark.parametrize("gate_norm", [0, 1])
def test_middle_at_the_edges_of_its_blocks(oracle, T, d, Hh, C, rows, gate_norm):
    _check(oracle, T, d, Hh, C, rows, gate_norm, 2)


# The tables are given, so T, k and the number of experts only say which form is taken: 64 expected rows and fewer, or many tiles, take
# the epilogue.  The last ones have 576 tiles, whose contraction is two k-tiles, whole or with a short one.
@pytest.mark.parametrize("T,d,Hh,C,rows,k,saved", [
    (400, 136, 64, 300, (0, 127, 128, 129, 255, 256, 257, 300), 1, True),
    (700, 264, 328, 640, (159, 160, 161, 512, 513, 640, 2, 64, 0, 1, 33), 1, False),
    (700, 128, 72, 640, (31, 640, 0, 257, 8, 9, 7, 384, 385, 65, 1), 1, True),
    (900, 128, 200, 8192, (0, 1, 255, 256, 257, 900) + (30,) * 9, 1, False),
    (420, 128, 4392, 400, (257, 300, 310, 400, 333, 288, 289, 260, 384, 385, 290, 352, 353, 399, 270, 320), 8, True),
    (420, 136, 4392, 400, (257, 300, 310, 400, 333, 288, 289, 260, 384, 385, 290, 352, 353, 399, 270, 320), 8, False)])
def test_middle_in_the_product(oracle, T, d, Hh, C, rows, k, saved):
    expected = min(C, -(-T * k // len(rows)))
    assert expected <= 64 or len(rows) * -(-expected // 256) * -(-Hh // 256) >= 128
    _check(oracle, T, d, Hh, C, rows, len(rows) & 1, k, saved)


def _check(oracle, T, d, Hh, C, rows, gate_norm, k, saved=False):
    import gpu_helpers as H
    B.load_library()
    E = len(rows)
    shape = I.EtrShape("middle", 43, T=T, d=d, E=E, D=8, k=k, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_BIDIR, recipe="iso",
                       n_centroids=E)
    print(f"backward middle T={T} d={d} H={Hh} C={C} rows={rows} gate_norm={gate_norm}", flush=True)
    L = H.GpuLayer(shape, gate_norm=gate_norm)
    L.route()
    kept = {}
    if saved:                                            # x W_gate and x W_up of the given rows, as the forward call keeps them
        kept = {n: torch.full((E, C, Hh), float("nan"), dtype=shape.torch_dtype, device="cuda") for n in ("a_saved", "b_saved")}
    slot_of, slot_token = np.full((T, E), -1, np.int32), np.full((E, C), -1, np.int32)
    rng = np.random.default_rng(5)
    for e, n in enumerate(rows):
        tokens = np.sort(rng.choice(T, n, replace=False))
        slot_token[e, :n] = tokens
        slot_of[tokens, e] = np.arange(n)
    tables = [torch.from_numpy(v).cuda() for v in (slot_of, slot_token, np.array(rows, np.int32))]
    dout = I.make_upstream_gradient(shape, "cuda")
    t = L.t
    for name, w in zip(kept, (t["w_gate"], t["w_up"])):
        for e, n in enumerate(rows):
            kept[name][e, :n] = (t["x"][tables[1][e, :n].long()].float() @ w[e].float().t()).to(shape.torch_dtype)
    out = [torch.full(s, 7.0, dtype=shape.torch_dtype, device="cuda") for s in ((T, d), (E, Hh, d), (E, Hh, d), (E, d, Hh))]
    dgate = torch.full((T, E), 7.0, device="cuda")
    ws = B.alloc_workspace(B.etr_backward_workspace_bytes(L.cfg))
    ws.fill_(0xFF)
    B.etr_moe_backward(L.cfg, t["x"], t["w_emb"], t["w_gate"], t["w_up"], t["w_down"], L.score, L.gate, *tables, dout, *out, ws, dgate=dgate, **kept)
    torch.cuda.synchronize()
    hx = L.host_inputs()
    ref = oracle.moe_backward(*(hx[n] for n in ("x", "w_emb", "w_gate", "w_up", "w_down")), slot_of, H.to_np(dout), D=8, dtype=shape.dtype,
                              gate_norm=gate_norm)
    tol = H.TOL_OUT[shape.dtype]
    for name, v in zip(("dx", "dw_gate", "dw_up", "dw_down"), out):
        a = oracle.to_f64(H.to_np(v), shape.dtype)
        assert np.isfinite(a).all() and H.scale_rel_err(a, ref[name]) <= tol, name
        if name != "dx":
            for e, n in enumerate(rows):                 # each expert on its own scale; no rows: exact zeros
                assert H.scale_rel_err(a[e], ref[name][e]) <= tol if n else not a[e].any(), (name, e)
    assert H.scale_rel_err(H.to_np(dgate).astype(np.float64), ref["dgate"]) <= tol
