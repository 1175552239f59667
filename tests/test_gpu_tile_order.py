"""Which workgroup takes which tile: masked launches tile by tile through all problems (of an XCD, or of the launch where the problems are no multiple of
8), problem by problem where many problems have few tiles each at D = 128 or nothing is masked, pairs of tiles in whole rounds only.  Every problem
of such launches against plain fp32 torch.  Tolerance: P and dS in bf16, fp32 sums; relative L2 <= 5e-3 for the gradients and the output."""
import pytest
import torch

from paper_2511_02043_amd import functional as fn

pytestmark = pytest.mark.gpu

# B, H, Hkv, S, D
SHAPES = [(1, 3, 3, 300, 64), (3, 8, 2, 391, 64), (2, 16, 16, 129, 64), (17, 8, 8, 700, 64), (3, 3, 3, 300, 128), (2, 8, 8, 513, 128),
          (24, 16, 16, 400, 128), (23, 15, 5, 333, 128), (40, 8, 8, 500, 128), (36, 8, 4, 130, 128)]


def _reference(q, k, v, dout, causal, window):
    x = [t.detach().float().requires_grad_(True) for t in (q, k, v)]
    rep = q.shape[1] // k.shape[1]
    kk, vv = (t.repeat_interleave(rep, 1) for t in x[1:])
    s = torch.matmul(x[0], kk.transpose(-1, -2).contiguous()) * q.shape[-1] ** -0.5
    if causal:
        i = torch.arange(q.shape[2], device=q.device)
        hidden = i[None, :] > i[:, None]
        if window is not None:
            hidden |= i[None, :] < i[:, None] - window
        s = s.masked_fill(hidden, float("-inf"))
    out = torch.matmul(torch.softmax(s, -1), vv)
    return (out,) + torch.autograd.grad(out, x, dout.float())


@pytest.mark.parametrize("mask", ["none", "causal", "window"])
@pytest.mark.parametrize("B,H,Hkv,S,D", SHAPES)
def test_every_problem(B, H, Hkv, S, D, mask):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(S)
    q, k, v, dout = (torch.randn(B, h, S, D, generator=gen, device="cuda:0").to(torch.bfloat16) for h in (H, Hkv, Hkv, H))
    x = [t.clone().requires_grad_(True) for t in (q, k, v)]
    window = 100 if mask == "window" else None
    out = fn.attention(*x, **({"causal": True} if mask == "causal" else {"window": window} if window else {}))
    got = (out,) + torch.autograd.grad(out, x, dout)
    for name, a, r in zip(("out", "dq", "dk", "dv"), (x.detach() for x in got), _reference(q, k, v, dout, mask != "none", window)):
        err = (a.float() - r.detach()).flatten(2).norm(dim=-1) / r.detach().flatten(2).norm(dim=-1)
        assert float(err.max()) <= 5e-3, (name, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("mask", ["prefix", "causal"])
@pytest.mark.parametrize("B,H,Hkv,Sq,Sk,D", [(64, 16, 16, 150, 150, 64), (3, 8, 2, 300, 391, 64), (40, 8, 8, 260, 130, 64), (7, 3, 3, 140, 333, 128), (24, 16, 4, 200, 300, 128)])
def test_masks_that_hide_nothing(B, H, Hkv, Sq, Sk, D, mask):
    """A prefix over all keys and rows behind all keys under a causal mask: the order of calls without a mask, and their results."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(Sq)
    q, k, v, dout = (torch.randn(B, h, s, D, generator=gen, device="cuda:0").to(torch.bfloat16) for h, s in ((H, Sq), (Hkv, Sk), (Hkv, Sk), (H, Sq)))
    x = [t.clone().requires_grad_(True) for t in (q, k, v)]
    out = fn.attention(*x, **({"prefix": Sk} if mask == "prefix" else {"causal": True, "q_offset": Sk - 1}))
    got = (out,) + torch.autograd.grad(out, x, dout)
    for name, a, r in zip(("out", "dq", "dk", "dv"), (x.detach() for x in got), _reference(q, k, v, dout, False, None)):
        err = (a.float() - r.detach()).flatten(2).norm(dim=-1) / r.detach().flatten(2).norm(dim=-1)
        assert float(err.max()) <= 5e-3, (name, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("B,H,Hkv,Sq,Sk,D", [(64, 16, 16, 150, 700, 64), (43, 11, 11, 270, 1300, 64), (64, 16, 4, 150, 300, 64)])
def test_chunks_of_rows_behind_many_keys(B, H, Hkv, Sq, Sk, D):
    """Many problems of few tiles that see nearly the same keys: side by side, and with heads that share them tile by tile."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(Sq)
    q, k, v, dout = (torch.randn(B, h, s, D, generator=gen, device="cuda:0").to(torch.bfloat16) for h, s in ((H, Sq), (Hkv, Sk), (Hkv, Sk), (H, Sq)))
    x = [t.clone().requires_grad_(True) for t in (q, k, v)]
    out = fn.attention(*x, causal=True, q_offset=Sk - Sq)
    got = (out,) + torch.autograd.grad(out, x, dout)
    full = torch.zeros(B, H, Sk - Sq, D, device="cuda:0", dtype=torch.bfloat16)
    want = _reference(torch.cat([full, q], 2), k, v, torch.cat([full, dout], 2), True, None)
    for name, a, r in zip(("out", "dq", "dk", "dv"), (x.detach() for x in got), (r.detach()[:, :, -a.shape[2]:] for r, a in zip(want, got))):
        err = (a.float() - r).flatten(2).norm(dim=-1) / r.flatten(2).norm(dim=-1)
        assert float(err.max()) <= 5e-3, (name, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("B,H,Hkv,S,D,mask", [
    (16, 16, 16, 1024, 128, "causal"), (17, 16, 8, 1000, 128, "prefix"), (32, 16, 16, 700, 64, "causal"), (2, 16, 16, 4096, 64, "causal"),     # pairs of tiles
    (2, 8, 2, 600, 128, "documents"), (3, 16, 2, 500, 128, "documents"), (16, 8, 8, 600, 64, "documents"), (3, 5, 5, 391, 128, "documents"),
    (5, 8, 4, 391, 64, "prefix"), (24, 16, 16, 400, 128, "prefix")])
def test_pairs_prefixes_and_documents(B, H, Hkv, S, D, mask):
    """Launches whose workgroups take a long and a short tile; prefix masks; documents alone, whose dK / dV and, at D = 128 with shared keys, dQ go
    problem by problem."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(S)
    q, k, v, dout = (torch.randn(B, h, S, D, generator=gen, device="cuda:0").to(torch.bfloat16) for h in (H, Hkv, Hkv, H))
    ids = torch.cumsum(torch.rand(B, S, generator=gen, device="cuda:0") < 0.01, 1).int()
    i = torch.arange(S, device="cuda:0")
    hidden = {"causal": i[None, :] > i[:, None], "prefix": (i[None, :] > i[:, None]) & (i[None, :] >= S // 3)}.get(mask)
    x = [t.clone().requires_grad_(True) for t in (q, k, v)]
    out = fn.attention(*x, **{"causal": {"causal": True}, "prefix": {"prefix": S // 3}, "documents": {"q_doc_ids": ids}}[mask])
    got = (out.detach(),) + torch.autograd.grad(out, x, dout)
    for b in range(0, B, 5):                         # problem after problem: the reference's scores are large
        y = [t[b:b + 1].detach().float().requires_grad_(True) for t in (q, k, v)]
        kk, vv = (t.repeat_interleave(H // Hkv, 1) for t in y[1:])
        s = torch.matmul(y[0], kk.transpose(-1, -2).contiguous()) * D ** -0.5
        s = s.masked_fill(hidden if hidden is not None else ids[b][None, :] != ids[b][:, None], float("-inf"))
        ref = torch.matmul(torch.softmax(s, -1), vv)
        for name, a, r in zip(("out", "dq", "dk", "dv"), got, (ref.detach(),) + torch.autograd.grad(ref, y, dout[b:b + 1].float())):
            err = (a[b:b + 1].float() - r).flatten(2).norm(dim=-1) / r.flatten(2).norm(dim=-1)
            assert float(err.max()) <= 5e-3, (name, b, int(err.argmax()), float(err.max()))
