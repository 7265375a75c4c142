"""fp32 layers whose token matrix is larger than a buffer descriptor's range (4 GiB): the products that fetch its rows, forward and
backward, take 64-bit addresses.  Expert choice keeps a few tokens from anywhere in the matrix; the layer's output and all its
gradients on those against the same in 64 bits, the input gradient of every other token zero."""
import pytest
import torch

from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,C,Hh", [(1_060_000, 1024, 4, 48, 72), (1_060_000, 1024, 8, 700, 520)])
def test_rows_beyond_four_gigabytes(T, d, E, C, Hh):
    import gpu_helpers as H
    B.load_library()
    print(f"fp32 wide T={T} d={d} E={E} C={C} H={Hh}", flush=True)
    cfg = B.make_config(I.EtrShape("wide", 1, T=T, d=d, E=E, D=64, k=1, capacity=C, H=Hh, dtype=I.DT_F32, mode=I.MODE_ECR, recipe="iso"))
    g = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *n: torch.randn(*n, device="cuda", generator=g)
    x, dout = rand(T, d), rand(T, d)
    w_emb, wg, wu, wd = rand(E, d // 64), 0.05 * rand(E, Hh, d), 0.05 * rand(E, Hh, d), 0.05 * rand(E, d, Hh)
    out, dx = torch.empty_like(x), torch.full_like(x, float("nan"))
    score, gate = torch.empty(T, E, device="cuda"), torch.empty(T, E, device="cuda")
    topk, slot_of, slot_token, counts = (torch.empty(n, dtype=torch.int32, device="cuda") for n in ((T, 1), (T, E), (E, C), (E,)))
    tables = dict(score=score, gate=gate, topk_expert=topk, slot_of=slot_of, slot_token=slot_token, counts=counts)
    B.etr_moe_forward(cfg, x, w_emb, wg, wu, wd, out, B.alloc_workspace(B.etr_workspace_bytes(cfg)), **tables)
    grads = [torch.empty_like(v) for v in (wg, wu, wd)]
    B.etr_moe_backward(cfg, x, w_emb, wg, wu, wd, score, gate, slot_of, slot_token, counts, dout, dx, *grads,
                       B.alloc_workspace(B.etr_backward_workspace_bytes(cfg)))
    torch.cuda.synchronize()
    assert int(slot_token.max()) > T // 2 and torch.all(counts == C)
    tokens = slot_token.flatten().long().unique()        # the router on the kept tokens: Eq. 4 lifted to R^d, softmax over the experts
    xs = x[tokens].double().requires_grad_()
    lift = w_emb.double().repeat_interleave(64, dim=1)
    weight = torch.softmax(torch.nn.functional.cosine_similarity(xs.unsqueeze(1), lift.unsqueeze(0), dim=2), dim=1)
    dweight, dxs = torch.zeros_like(weight), torch.zeros_like(xs)
    expected = {}
    for e in range(E):
        t = slot_token[e].long()
        xe, go, w = x[t].double(), dout[t].double(), gate[t, e].double().unsqueeze(1)
        a, b = xe @ wg[e].double().t(), xe @ wu[e].double().t()
        sig = torch.sigmoid(a)
        h = a * sig * b
        y = w * (h @ wd[e].double().t())
        for i, token in enumerate(t.tolist()):
            expected[token] = expected[token] + y[i] if token in expected else y[i]
        dweight[torch.searchsorted(tokens, t), e] = (go * (h @ wd[e].double().t())).sum(1)
        dh = (w * go) @ wd[e].double()
        da, db = dh * b * sig * (1 + a * (1 - sig)), dh * a * sig
        dxs.index_add_(0, torch.searchsorted(tokens, t), da @ wg[e].double() + db @ wu[e].double())
        for got, ref in zip(grads, (da.t() @ xe, db.t() @ xe, (w * go).t() @ h)):
            assert (got[e].double() - ref).abs().max() <= H.TOL_OUT[I.DT_F32] * ref.abs().max(), e
    at = torch.tensor(list(expected), device="cuda")
    ref = torch.stack(list(expected.values()))
    assert (out[at].double() - ref).abs().max() <= H.TOL_OUT[I.DT_F32] * ref.abs().max()
    weight.backward(dweight)
    ref = dxs.detach() + xs.grad
    assert (dx[tokens].double() - ref).abs().max() <= H.TOL_OUT[I.DT_F32] * ref.abs().max()
    dx[tokens] = 0.0
    assert torch.all(dx.abs().amax(dim=1) == 0)          # (a NaN that nobody wrote over is not 0)
