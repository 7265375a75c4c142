"""The one-launch selection of short batches: token counts around whole waves and its limit, every mode, ties, capacities
below, at and above the candidates, a capacity read from the device, E with and without 16-byte rows."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,C,levels", [(1, 1, 1, 3, None), (2, 64, 3, 1, 2), (63, 5, 2, 20, 3), (64, 16, 16, 64, None),
                                            (65, 8, 1, 4, 5), (300, 33, 4, 25, 40), (511, 4, 2, 700, None), (512, 12, 3, 100, 9),
                                            (513, 12, 3, 100, 9)])
def test_small_select(oracle, T, E, k, C, levels):
    B.load_library()
    rng = np.random.default_rng(100 * T + E)
    S = (rng.integers(-levels, levels + 1, size=(T, E)) / levels if levels else rng.uniform(-1, 1, (T, E))).astype(np.float32)
    S[rng.random((T, E)) < 0.05] = -0.0
    Sd = torch.from_numpy(S).cuda()
    for mode in range(5):
        for cap in (None, max(1, C // 3)):
            cfg = B.make_config(I.EtrShape("s", 1, T=T, d=8 * E, E=E, D=8, k=k, capacity=C, H=8, dtype=I.DT_F32, mode=mode,
                                           recipe="iso"))
            topk, slot_of, slot_token, counts = (torch.full(n, -7, dtype=torch.int32, device="cuda")
                                                 for n in ((T, k), (T, E), (E, C), (E,)))
            ws = B.alloc_workspace(B.etr_select_workspace_bytes(cfg))
            if cap is None:
                B.etr_select(cfg, Sd, topk, slot_of, slot_token, counts, ws)
            else:
                B.etr_select_adaptive(cfg, Sd, torch.tensor([cap], dtype=torch.int32, device="cuda"), 0.0, topk, slot_of,
                                      slot_token, counts, ws)
            torch.cuda.synchronize()
            o_tk, o_so, o_st, o_c = oracle.select(S, k, cap or C, mode)
            np.testing.assert_array_equal(counts.cpu().numpy(), o_c)
            np.testing.assert_array_equal(slot_of.cpu().numpy(), o_so)
            st = slot_token.cpu().numpy()
            np.testing.assert_array_equal(st[:, :cap or C], o_st)
            assert np.all(st[:, cap or C:] == -1)
            if mode == I.MODE_ECR:
                assert torch.all(topk == -7)
            else:
                np.testing.assert_array_equal(topk.cpu().numpy(), o_tk)


@pytest.mark.parametrize("T,E,k,C,levels", [(64, 8, 6, 30, 7), (65, 8, 7, 30, None), (200, 12, 10, 150, 5), (512, 64, 48, 380, None),
                                            (512, 64, 49, 200, 9), (511, 8, 8, 100, None), (16, 4, 3, 9, None)])
def test_small_select_around_three_quarters(oracle, T, E, k, C, levels):
    """Experts kept by most of the tokens: candidates counted where they lie and brought together, the second again with an affinity
    sum that ends inside the list, reaches its end, or is beyond it."""
    test_small_select(oracle, T, E, k, C, levels)
    rng = np.random.default_rng(T + E)
    S = (rng.integers(-levels, levels + 1, size=(T, E)) / levels if levels else rng.uniform(-1, 1, (T, E))).astype(np.float32)
    Sd = torch.from_numpy(S).cuda()
    for mode in (I.MODE_ECR, I.MODE_BIDIR):
        for thr in (0.2 * T * 0.3, 0.9 * T * 0.3, 10.0 * T):
            cfg = B.make_config(I.EtrShape("s", 1, T=T, d=8 * E, E=E, D=8, k=k, capacity=C, H=8, dtype=I.DT_F32, mode=mode, recipe="iso"))
            topk, slot_of, slot_token, counts = (torch.full(n, -7, dtype=torch.int32, device="cuda") for n in ((T, k), (T, E), (E, C), (E,)))
            B.etr_select_adaptive(cfg, Sd, None, float(np.float32(thr)), topk, slot_of, slot_token, counts,
                                  B.alloc_workspace(B.etr_select_workspace_bytes(cfg)))
            torch.cuda.synchronize()
            _, o_so, o_st, o_c = oracle.select_adaptive(S, k, C, mode, float(np.float32(thr)))
            np.testing.assert_array_equal(counts.cpu().numpy(), o_c)
            np.testing.assert_array_equal(slot_of.cpu().numpy(), o_so)
            st = slot_token.cpu().numpy()
            np.testing.assert_array_equal(st[:, :o_st.shape[1]], o_st)
            assert np.all(st[:, o_st.shape[1]:] == -1)
