"""The bf16 GEMM for few rows per expert: one, two and four 16-row blocks, several row blocks of 64, empty experts,
contractions of less than one chunk, of whole chunks and ragged ones, narrow and ragged outputs; in
the forward, the training forward and the recomputation of the backward."""
import numpy as np
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,C,d,Hh,counts", [
    (4, 16, 2048, 1024, [16, 1, 0, 15]),                 # one block of 16 rows; 16 and 8 chunks of k
    (3, 33, 1080, 520, [33, 17, 32]),                    # two blocks and one past; short last chunks
    (64, 64, 136, 40, [64, 0, 49, 1] * 16),              # one whole chunk and a short one; outputs narrower than a workgroup's
    (2, 30, 8, 8, [30, 3]),                              # less than one k-step
    (4, 64, 56, 1024, [64, 17, 0, 16]),                  # less than one k-tile, many columns; then eight chunks
    (1, 200, 320, 4096, [200]),                          # four row blocks, the last of 8 rows; two whole chunks and a half one
    (5, 64, 192, 72, [64, 63, 48, 31, 0]),
])
def test_few_rows_ffn(oracle, E, C, d, Hh, counts):
    import gpu_helpers as H
    import test_gpu_parity
    B.load_library()
    # (that test's layers have T = C tokens on one expert each: C / E rows are expected, which chooses this kernel)
    cfg = B.make_config(I.EtrShape("f", 1, T=C, d=d, E=E, D=8, k=1, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_TCR,
                                   recipe="iso"))
    assert [H.ffn_plan(cfg, p, gathered=False)[0] for p in (0, 1)] == [H.ROWS, H.ROWS]
    test_gpu_parity.test_expert_ffn(H, oracle, I.DT_BF16, E, C, d, Hh, counts)


@pytest.mark.parametrize("T,d,Hh,E,k,mode", [(1, 256, 512, 8, 2, I.MODE_TCR), (7, 264, 136, 4, 4, I.MODE_BIDIR),
                                             (100, 512, 328, 6, 2, I.MODE_BIDIR), (150, 1024, 256, 16, 1, I.MODE_ECR)])
def test_few_rows_layer_and_backward(oracle, T, d, Hh, E, k, mode):
    import gpu_helpers as H
    from test_gpu_backward import Backward, _err
    B.load_library()
    C = T if mode != I.MODE_ECR else 12
    shape = I.EtrShape("few", 12, T=T, d=d, E=E, D=8, k=k, capacity=C, H=Hh, dtype=I.DT_BF16, mode=mode, recipe="bias")
    print(f"few rows T={T} d={d} H={Hh} E={E} k={k} mode={mode}", flush=True)
    L = H.GpuLayer(shape)
    assert [H.ffn_plan(L.cfg, p)[0] for p in (0, 1)] == [H.ROWS, H.ROWS]
    hx = L.host_inputs()
    L.forward()
    r = H.check_routing_against_oracle(oracle, L, hx)
    H.check_output_against_oracle(oracle, L, hx, r["score"])
    bw = Backward(H, shape, mode)
    hb = bw.host()
    ref = oracle.moe_backward(hb["x"], hb["w_emb"], hb["w_gate"], hb["w_up"], hb["w_down"], hb["slot_of"], hb["dout"],
                              D=shape.D, dtype=shape.dtype)
    for got, key in ((bw.dx, "dx"), (bw.dwg, "dw_gate"), (bw.dwu, "dw_up"), (bw.dwd, "dw_down")):
        assert _err(H, oracle, got, ref[key], shape.dtype) <= H.TOL_OUT[shape.dtype], key
    # kept and recomputed pre-activations come from the same kernel: the same bits through the backward
    t, cfg = L.t, L.cfg
    a, b = (torch.empty(E, C, Hh, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    out = torch.empty_like(L.out)
    B.etr_moe_forward_train(cfg, t["x"], t["w_emb"], t["w_gate"], t["w_up"], t["w_down"], out, a, b,
                            B.alloc_workspace(B.etr_workspace_bytes(cfg)))
    dx, dwg, dwu, dwd = (torch.empty_like(v) for v in (bw.dx, bw.dwg, bw.dwu, bw.dwd))
    B.etr_moe_backward(cfg, t["x"], t["w_emb"], t["w_gate"], t["w_up"], t["w_down"], bw.L.score, bw.L.gate, bw.L.slot_of,
                       bw.L.slot_token, bw.L.counts, bw.dout, dx, dwg, dwu, dwd,
                       B.alloc_workspace(B.etr_backward_workspace_bytes(cfg)), a_saved=a, b_saved=b)
    torch.cuda.synchronize()
    assert torch.equal(out, L.out)
    for got, want in ((dx, bw.dx), (dwg, bw.dwg), (dwu, bw.dwu), (dwd, bw.dwd)):
        assert np.array_equal(H.to_np(got), H.to_np(want))


@pytest.mark.parametrize("T,E,C,d,Hh,counts", [
    (8, 4, 300, 512, 1024, [300, 0, 129, 64]),           # five row tiles and more, a grid for four experts' partial ones
    (3, 2, 1000, 512, 520, [1000, 1000]),
    (70, 64, 200, 256, 512, [200, 1, 0, 65] * 16),
])
def test_counts_beyond_the_batch(oracle, T, E, C, d, Hh, counts):
    """The stage call on rows that other processes sent: the counts exceed what this config's tokens could fill, so every
    workgroup takes several tiles."""
    import gpu_helpers as H
    B.load_library()
    print(f"counts beyond the batch T={T} E={E} C={C} d={d} H={Hh}", flush=True)
    shape = I.EtrShape("ep", 1, T=T, d=d, E=E, D=8, k=1, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_BIDIR, recipe="iso")
    cfg = B.make_config(shape)
    for product, cols in ((0, 32), (1, 64)):
        kernel, groups = H.ffn_plan(cfg, product, gathered=False)
        assert kernel == H.ROWS
        assert groups < sum(-(-n // 64) for n in counts) * -(-(d if product else Hh) // cols)
    H.check_expert_ffn(oracle, shape, counts)


@pytest.mark.parametrize("E,C,d,Hh", [(16, 700, 2048, 1024), (16, 520, 512, 1408), (64, 300, 320, 512), (16, 700, 1032, 1048),
                                      (32, 700, 1048, 184)])
def test_same_bits_as_many_rows(E, C, d, Hh):
    """The few-rows kernel adds the products in the order of the persistent one: the same rows give the same bits whichever
    of the two a batch takes."""
    import gpu_helpers as H
    B.load_library()
    print(f"same bits E={E} C={C} d={d} H={Hh}", flush=True)
    dt = torch.bfloat16
    xp = I.normal(1, E * C * d, "cuda").reshape(E, C, d).to(dt)
    wg, wu = (I.ffn_weight(s, (E, Hh, d), dt, "cuda", std=0.05) for s in (2, 3))
    wd = I.ffn_weight(4, (E, d, Hh), dt, "cuda", std=0.05)
    counts = torch.tensor([max(0, C - 37 * e) if e != 1 else 0 for e in range(E)], dtype=torch.int32, device="cuda")
    out, hidden, kernels = [], [], []
    for T in (1, 64 * 4096):
        cfg = B.make_config(I.EtrShape("b", 1, T=T, d=d, E=E, D=8, k=1, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_BIDIR,
                                       recipe="iso"))
        kernels.append([H.ffn_plan(cfg, p, gathered=False)[0] for p in (0, 1)])
        ws = torch.zeros(B.etr_ffn_workspace_bytes(cfg) // 2, dtype=dt, device="cuda")
        yp = torch.zeros(E, C, d, dtype=dt, device="cuda")
        B.etr_expert_ffn(cfg, xp, counts, wg, wu, wd, yp, ws)
        torch.cuda.synchronize()
        out.append(yp)
        hidden.append(ws[:E * C * Hh])                   # the scratch is the hidden activation
    assert kernels[0] == [H.ROWS, H.ROWS]
    assert kernels[1] == [H.PERSISTENT if n % 64 == 0 else H.PERSISTENT_TAIL for n in (d, Hh)]
    live = torch.arange(C, device="cuda").unsqueeze(0) < counts.unsqueeze(1)
    assert torch.equal(hidden[0].view(E, C, Hh)[live], hidden[1].view(E, C, Hh)[live])
    assert torch.equal(out[0], out[1])


_P, _Z, _R = "PERSISTENT", "PERSISTENT_TAIL", "ROWS"


@pytest.mark.parametrize("E,C,d,Hh,kernels,counts", [
    (6, 900, 768, 1152, (_P, _P), [900, 0, 513, 1, 899, 256]),
    (16, 1100, 256, 2816, (_P, _P), [1100, 700, 1, 1024, 0, 1025, 300, 1100] * 2),
    (8, 2048, 128, 1024, (_P, _R), [2048, 1500, 2048, 300, 2047, 1025, 2048, 1800]),     # two k-tiles; a narrow output
    (8, 2048, 2048, 128, (_P, _P), [2048, 1500, 0, 300, 2047, 1025, 2048, 1800]),
    (2, 4200, 1024, 384, (_P, _P), [4200, 3333]),
    (16, 520, 1080, 1320, (_Z, _Z), [520, 513, 0, 3] * 4),               # both contractions end 56 and 40 past whole k-tiles
    (16, 700, 1032, 1048, (_Z, _Z), [700, 0, 257, 256, 255, 1, 128, 300] * 2),           # 8 and 24 past
    # three k-tiles, the third short: its token rows are the first copies behind the prologue, its weight rows follow a
    # k-tile later, and a workgroup's second tile starts inside that; gate/up, then down
    (16, 1100, 136, 1048, (_Z, None), [1100, 0, 1025, 769, 1, 512, 1100, 300] * 2),
    (16, 1100, 184, 1048, (_Z, None), [1100, 0, 1025, 769, 1, 512, 1100, 300] * 2),
    (32, 700, 1048, 136, (None, _Z), [700, 0, 513, 256, 1, 512, 699, 300] * 4),
    (32, 700, 1048, 184, (None, _Z), [700, 0, 513, 256, 1, 512, 699, 300] * 4),
    # the kernels with a workgroup per tile: outputs too narrow for the persistent one; ragged and small
    (16, 3000, 128, 64, ("RING", "RING"), [3000, 0, 2049, 1, 256, 257, 1025, 2999] * 2),
    (16, 300, 1032, 1048, ("STAGED", "STAGED"), [300, 0, 257, 256, 255, 1, 128, 300] * 2),
])
def test_many_rows_expected_ffn(oracle, E, C, d, Hh, kernels, counts):
    """The same stage where every expert is expected to fill its capacity: mostly the 256-row tiles of the persistent kernel,
    on ragged counts, contractions and column tails."""
    import gpu_helpers as H
    B.load_library()
    print(f"ffn with {E} x {C} rows expected, d={d} H={Hh}", flush=True)
    shape = I.EtrShape("m", 1, T=E * C, d=d, E=E, D=8, k=1, capacity=C, H=Hh, dtype=I.DT_BF16, mode=I.MODE_TCR, recipe="iso")
    for product, kernel in enumerate(kernels):
        if kernel:
            assert H.ffn_plan(B.make_config(shape), product, gathered=False)[0] == getattr(H, kernel)
    H.check_expert_ffn(oracle, shape, counts)
