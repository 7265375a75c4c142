"""Routing with large embeddings, where the waves of a workgroup that share one copy of them are chosen by what fits a CU: 4, 8
and 16 waves, both sides of the token count from which more than 4 are taken, pooled features that the dot product's steps do
and do not divide, rows of one and of several passes.  Scores and gates against the oracle with the layer's tolerance."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu

# (T, d, E, D, dtype, cos); pooled features, waves on 256 CUs
CASES = [
    (900, 4096, 64, 8, I.DT_BF16, I.COS_FULL),       # 512: 4 (one workgroup to a CU, every token resident)
    (1500, 4096, 64, 8, I.DT_BF16, I.COS_POOLED),    # 512: 8
    (2500, 4096, 32, 8, I.DT_BF16, I.COS_FULL),      # 512: 16
    (2301, 4096, 64, 16, I.DT_BF16, I.COS_FULL),     # 256: 8
    (3200, 3840, 48, 16, I.DT_BF16, I.COS_FULL),     # 240: 8, lanes without an expert
    (2200, 2048, 64, 8, I.DT_F32, I.COS_POOLED),     # 256: 8
    (2300, 2056, 64, 8, I.DT_BF16, I.COS_FULL),      # 257: 8, one feature at a time
    (3100, 4080, 64, 24, I.DT_BF16, I.COS_POOLED),   # 170: 8, a lane per pooled feature
    (1100, 8192, 64, 16, I.DT_BF16, I.COS_FULL),     # 512: 8, two passes over a row
    (40, 1072, 5, 8, I.DT_BF16, I.COS_FULL),         # 134: 4, eight lanes to an expert
]


@pytest.mark.parametrize("T,d,E,D,dtype,cos", CASES)
def test_route(oracle, T, d, E, D, dtype, cos):
    import gpu_helpers as H
    B.load_library()
    shape = I.EtrShape("route", 29, T=T, d=d, E=E, D=D, k=1, capacity=T, H=64, dtype=dtype, mode=I.MODE_BIDIR, recipe="iso",
                       cos=cos)
    print(f"route T={T} d={d} E={E} D={D} dtype={dtype} cos={cos}", flush=True)
    gen = torch.Generator().manual_seed(29)
    x = (torch.randn(T, d, generator=gen) + 0.5 * torch.randn(T, 1, generator=gen)).to(shape.torch_dtype).cuda()
    w = torch.randn(E, d // D, generator=gen).cuda()
    score = torch.full((T, E), float("nan"), device="cuda")
    gate = torch.full((T, E), float("nan"), device="cuda")
    B.etr_route(B.make_config(shape), x, w, score, gate)
    torch.cuda.synchronize()
    ref_score, ref_gate = oracle.route(H.to_np(x), w.cpu().numpy(), D, dtype, cos)[:2]
    assert np.max(np.abs(score.cpu().numpy() - ref_score)) <= H.TOL_SCORE
    assert np.max(np.abs(gate.cpu().numpy() - ref_gate)) <= H.TOL_GATE
