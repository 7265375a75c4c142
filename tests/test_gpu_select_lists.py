"""The selection by lists of the chosen pairs: token counts around whole tiles and its limits, rows of scores with and without 16-byte
pieces, one to four experts a token, every expert or one expert chosen by all (more pairs than the column's room in LDS), ties,
capacities that turn nobody, some and nearly all away, a capacity read from the device, affinity sums.  The tables of the oracle."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


def _scores(kind, T, E):
    rng = np.random.default_rng(T + 7 * E)
    s = rng.uniform(-1, 1, (T, E)).astype(np.float32)
    if kind == "ties":
        s = (np.round(s * 3) / 3).astype(np.float32)
        s[rng.random((T, E)) < 0.05] = -0.0
    if kind == "one":                                    # the first expert is everybody's choice
        s = s * np.float32(0.01)
        s[:, 0] = rng.uniform(0.2, 0.3, T).astype(np.float32)
    if kind == "copies":                                 # half of the tokens are one token, with two experts far ahead
        s[rng.random(T) < 0.5] = np.where(np.arange(E) < 2, np.float32(0.9), s[0] * np.float32(0.1)).astype(np.float32)
    if kind == "half":                                   # half of the tokens on one expert, a quarter on the next, ...
        s *= np.float32(0.05)
        s[np.arange(T), rng.geometric(0.5, T).clip(1, E) - 1] += np.float32(0.5)
    return s


@pytest.mark.parametrize("T,E,k,kind", [(1025, 8, 1, "any"), (1088, 64, 4, "ties"), (1089, 13, 3, "any"), (2047, 33, 2, "ties"), (4096, 32, 4, "one"),
                                        (9001, 12, 1, "any"), (40000, 8, 1, "one"), (65536, 16, 2, "one"), (65536, 63, 4, "any"), (65537, 8, 1, "any"),
                                        (3000, 4, 1, "ties")])
def test_selection_by_lists(oracle, T, E, k, kind):
    B.load_library()
    S = _scores(kind, T, E)
    Sd = torch.from_numpy(S).cuda()
    even = max(1, T * k // E)
    pos = float(np.sort(np.maximum(S.astype(np.float64), 0), axis=1)[:, -k:].sum()) / E
    for mode in (I.MODE_TCR, I.MODE_BIDIR, 3):           # 3: first choices before second ones
        for C, cap, thr in ((even, None, 0.0), (T, None, 0.0), (max(1, even // 7), None, 0.0), (even, max(1, even // 3), 0.0), (T, None, 0.4 * pos),
                            (even, None, 2 * pos + 1)):
            if thr and mode != I.MODE_BIDIR:
                continue
            print(f"select lists T={T} E={E} k={k} {kind} mode={mode} C={C} cap={cap} thr={thr:.4g}", flush=True)
            cfg = B.make_config(I.EtrShape("l", 1, T=T, d=8 * E, E=E, D=8, k=k, capacity=C, H=8, dtype=I.DT_F32, mode=mode, recipe="iso"))
            topk, slot_of, slot_token, counts = (torch.full(n, -7, dtype=torch.int32, device="cuda") for n in ((T, k), (T, E), (E, C), (E,)))
            ws = B.alloc_workspace(B.etr_select_workspace_bytes(cfg))
            ws.fill_(0xFF)
            if cap is None and not thr:
                B.etr_select(cfg, Sd, topk, slot_of, slot_token, counts, ws)
                ref = oracle.select(S, k, C, mode)
            else:
                dev = None if cap is None else torch.tensor([cap], dtype=torch.int32, device="cuda")
                B.etr_select_adaptive(cfg, Sd, dev, float(np.float32(thr)), topk, slot_of, slot_token, counts, ws)
                ref = oracle.select_adaptive(S, k, C, mode, float(np.float32(thr))) if thr else oracle.select(S, k, cap, mode)
            torch.cuda.synchronize()
            o_tk, o_so, o_st, o_c = ref
            np.testing.assert_array_equal(counts.cpu().numpy(), o_c)
            np.testing.assert_array_equal(slot_of.cpu().numpy(), o_so)
            st = slot_token.cpu().numpy()
            np.testing.assert_array_equal(st[:, :o_st.shape[1]], o_st)
            assert np.all(st[:, o_st.shape[1]:] == -1)
            np.testing.assert_array_equal(topk.cpu().numpy(), o_tk)


@pytest.mark.parametrize("T,E,k,kind", [(1100, 8, 2, "half"), (2048, 8, 2, "copies"), (4097, 16, 4, "half"), (8192, 16, 2, "one"), (8193, 16, 4, "copies"),
                                        (16384, 32, 4, "half"), (20000, 8, 2, "copies"), (32768, 16, 4, "half"), (32769, 64, 4, "copies"),
                                        (65536, 8, 1, "half"), (65500, 12, 3, "copies"), (65536, 64, 1, "one"),
                                        (16300, 8, 2, "any"), (32700, 9, 2, "ties"), (49152, 8, 2, "half")])
def test_crowded_columns(oracle, T, E, k, kind):
    """Columns that stay in registers, of every length: thresholds inside a run of equal keys, with and without an affinity sum."""
    test_selection_by_lists(oracle, T, E, k, kind)


def test_capture_behind_a_first_call_at_another_shape(oracle):
    """Captured calls without a first call at their shape, with a threshold and without: replays on other scores."""
    B.load_library()
    print("select lists under capture", flush=True)
    small = B.make_config(I.EtrShape("s", 1, T=100, d=64, E=8, D=8, k=1, capacity=20, H=8, dtype=I.DT_F32, mode=I.MODE_BIDIR, recipe="iso"))
    tables = lambda T, E, C, k: [torch.full(n, -7, dtype=torch.int32, device="cuda") for n in ((T, k), (T, E), (E, C), (E,))]
    B.etr_select_noalloc(small, torch.rand(100, 8, device="cuda"), *tables(100, 8, 20, 1))
    T, E, k, C = 3500, 20, 2, 200
    cfg = B.make_config(I.EtrShape("l", 1, T=T, d=8 * E, E=E, D=8, k=k, capacity=C, H=8, dtype=I.DT_F32, mode=I.MODE_BIDIR, recipe="iso"))
    score, plain, summed = torch.zeros(T, E, device="cuda"), tables(T, E, C, k), tables(T, E, C, k)
    ws = B.alloc_workspace(B.etr_select_workspace_bytes(cfg))
    thr = 20.0
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        B.etr_select_noalloc(cfg, score, *plain)
        B.etr_select_adaptive(cfg, score, None, thr, *summed, ws)
    for rep in range(3):
        S = np.roll(_scores("any", T, E), rep, axis=1)
        score.copy_(torch.from_numpy(S))
        for t in plain + summed:
            t.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in ((plain, oracle.select(S, k, C, I.MODE_BIDIR)), (summed, oracle.select_adaptive(S, k, C, I.MODE_BIDIR, thr))):
            for t, o in zip(got, ref):
                a = t.cpu().numpy()
                np.testing.assert_array_equal(a[:, :o.shape[1]] if o.ndim == 2 else a, o)
                assert o.ndim == 1 or np.all(a[:, o.shape[1]:] == -1)
