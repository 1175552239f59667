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


def _forward(q, k, v, cap, mask):
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device=q.device)
    lse = torch.full(q.shape[:-1] + (1,), float("nan"), dtype=torch.float32, device=q.device)
    desc = fb.variant_desc(scale=q.shape[-1] ** -0.5, score_mod=fb.FL_MOD_SOFTCAP, softcap=cap, mask=mask)
    fb.check(fb.fl_attn_fwd(*(fb.tensor_desc(x) for x in (q, k, v)), desc, None, fb.tensor_desc(out), fb.tensor_desc(lse),
                            torch.cuda.current_stream().cuda_stream))
    return out, lse[..., 0]


def _inputs(S, D):
    gen = torch.Generator(device="cuda:0").manual_seed(S + D)
    return [(3.0 * torch.randn(2, 1, 2, S, D, generator=gen, device="cuda:0")).to(torch.bfloat16) for _ in range(3)]


@pytest.mark.parametrize("cap", [1e-3, 1.0, 30.0, 1e4])
@pytest.mark.parametrize("D", [64, 128])
def test_largest_score_has_probability_one(cap, D):
    """A row's reference is its largest score, without a rounding between the two: a row with a single visible key gives that key's
    values, to the bit."""
    q, k, v = _inputs(70, D)
    out, _ = _forward(q, k, v, cap, fb.FL_MASK_CAUSAL)
    assert torch.equal(out[..., 0, :], v[..., 0, :].float())


@pytest.mark.parametrize("cap", [1.5e-45, 1e-38, 1e30, 3e38])
def test_extreme_caps(cap):
    """Caps so small or so large that every capped score is 0 in fp32: the mean of V (P = 1 exactly; sums of S bf16 values in fp32)."""
    q, k, v = _inputs(100, 64)
    out, lse = _forward(q, k, v, cap, 0)
    ref = v.double().mean(-2, keepdim=True).expand(out.shape)
    assert float((out.double() - ref).norm() / ref.norm()) <= 100 * 2.0 ** -24
    assert float((lse.double() - torch.log(torch.tensor(100.0)).item()).abs().max()) <= 1e-5
