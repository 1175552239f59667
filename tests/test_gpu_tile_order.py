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
