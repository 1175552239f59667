"""Soft-capped scores over the range of caps: output and saved log-sum-exp against an fp64 evaluation.

Bounds.  Output: bf16 probabilities, 2^-9 relative L2 (1.7e-3 measured), bound 5e-3.  lse: a capped score is cap * (1 - 2 t) with
t = 1 / (exp(2 z) + 1) in fp32, three roundings of 2^-23 at most, so it is off by at most 6 * 2^-23 * cap <= cap * 2^-20; the sums
and the logarithm add 1e-5."""
import pytest
import torch

from paper_2511_02043_amd import binding as fb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [1e-3, 1.0, 30.0, 1e4])
@pytest.mark.parametrize("D,S,mask", [(64, 1, 0), (64, 333, 0), (64, 1025, fb.FL_MASK_CAUSAL), (128, 257, 0), (128, 129, fb.FL_MASK_CAUSAL)])
def test_soft_cap(cap, D, S, mask):
    gen = torch.Generator(device="cuda:0").manual_seed(S + D)
    q, k, v = ((3.0 * torch.randn(2, 1, 2, S, D, generator=gen, device="cuda:0")).to(torch.bfloat16) for _ in range(3))
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device=q.device)
    lse = torch.full(q.shape[:-1] + (1,), float("nan"), dtype=torch.float32, device=q.device)
    desc = fb.variant_desc(scale=D ** -0.5, score_mod=fb.FL_MOD_SOFTCAP, softcap=cap, mask=mask)
    fb.check(fb.fl_attn_fwd(*(fb.tensor_desc(x) for x in (q, k, v)), desc, None, fb.tensor_desc(out), fb.tensor_desc(lse),
                            torch.cuda.current_stream().cuda_stream))
    s = q.double() @ k.double().transpose(-1, -2).contiguous() * D ** -0.5
    s = cap * torch.tanh(s / cap)
    if mask:
        s = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device=s.device).triu(1), -float("inf"))
    ref = torch.softmax(s, -1) @ v.double()
    err = float((out.double() - ref).norm() / ref.norm())
    lse_err = float((lse[..., 0].double() - torch.logsumexp(s, -1)).abs().max())
    print(f"cap {cap} D {D} S {S}: rel {err:.2e} lse {lse_err:.2e}", flush=True)
    assert err <= 5e-3
    assert lse_err <= cap * 2.0 ** -20 + 1e-5
