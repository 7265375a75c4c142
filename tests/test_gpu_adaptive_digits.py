"""The adaptive token count: by counting in the one-launch selection of short batches, and its digit-by-digit threshold
search at every chunk length of the per-expert kernel (registers, slice histograms, streamed columns), on affinities that crowd into few digits, tie, or round to zero terms; and the
routing statistics at token counts around the unrolled pass of a workgroup."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


def _scores(kind, T, E):
    rng = np.random.default_rng(T + 13 * E)
    s = rng.standard_normal((T, E)).astype(np.float32)
    if kind == "cosine":                                 # what routing gives: small, both signs
        return s * np.float32(0.016)
    if kind == "crowded":                                # one exponent, few distinct mantissas
        return np.float32(0.5) + np.round(np.abs(s) * 4).astype(np.float32) * np.float32(2.0 ** -22)
    s = np.where(rng.random((T, E)) < 0.7, np.abs(s) * np.float32(1e-11), s * np.float32(0.1))   # "zeros": terms of 0
    s[rng.random((T, E)) < 0.01] = 1.0
    return s.astype(np.float32)


@pytest.mark.parametrize("T,E,k", [(1, 2, 1), (130, 7, 3), (512, 4, 2), (900, 3, 2), (8000, 2, 1), (15000, 5, 2), (32768, 2, 2), (65536, 33, 4), (66001, 3, 1)])
@pytest.mark.parametrize("kind", ["cosine", "crowded", "zeros"])
def test_adaptive_count_digits(oracle, T, E, k, kind):
    B.load_library()
    S = _scores(kind, T, E)
    Sd = torch.from_numpy(S).cuda()
    pos = float(np.maximum(S.astype(np.float64), 0).sum()) / E
    for mode, thr in ((I.MODE_ECR, 0.3 * pos), (I.MODE_BIDIR, 0.1 * pos * k / E), (I.MODE_ECR, 1e-9), (I.MODE_BIDIR, 4 * pos + 1)):
        print(f"adaptive digits T={T} E={E} k={k} {kind} mode={mode} thr={thr:.4g}", flush=True)
        C = T
        cfg = B.make_config(I.EtrShape("a", 1, T=T, d=8 * E, E=E, D=8, k=k, capacity=C, H=8, dtype=I.DT_F32, mode=mode,
                                       recipe="iso"))
        slot_of, slot_token, counts = (torch.empty(*n, dtype=torch.int32, device="cuda") for n in ((T, E), (E, C), (E,)))
        topk = torch.empty(T, k, dtype=torch.int32, device="cuda")
        B.etr_select_adaptive(cfg, Sd, None, float(np.float32(thr)), topk, slot_of, slot_token, counts,
                              B.alloc_workspace(B.etr_select_workspace_bytes(cfg)))
        torch.cuda.synchronize()
        o_tk, o_so, o_st, o_c = oracle.select_adaptive(S, k, C, mode, float(np.float32(thr)))
        np.testing.assert_array_equal(counts.cpu().numpy(), o_c)
        np.testing.assert_array_equal(slot_of.cpu().numpy(), o_so)
        if mode != I.MODE_ECR:
            np.testing.assert_array_equal(topk.cpu().numpy(), o_tk)


@pytest.mark.parametrize("T,E,k", [(1, 64, 1), (31, 64, 2), (257, 33, 2), (8193, 3, 1), (300000, 8, 2)])
def test_route_stats_token_counts(oracle, T, E, k):
    import test_gpu_stats
    B.load_library()
    test_gpu_stats.test_route_stats(oracle, T, E, k, max(1, T * k // (2 * E)), I.MODE_BIDIR)
