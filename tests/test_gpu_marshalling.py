"""The compiled marshalling of the PyTorch entry points: 4-D and 5-D tensors, strided views, an expanded output gradient and a
caller's workspace reach the C ABI as the tensors they are, and what it does not take is refused before a launch."""
import pytest
import torch

from paper_2511_02043_amd import functional as F

pytestmark = pytest.mark.gpu


def normal(*shape, seed=0):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    return torch.randn(shape, generator=gen, device="cuda:0").bfloat16()


def grads(q, k, v, **kw):
    x = [t.detach().requires_grad_(True) for t in (q, k, v)]
    out = F.attention(*x, **kw)
    return (out.detach(),) + torch.autograd.grad(out.sum(), x)      # (the gradient of a sum arrives as an expanded scalar)


def test_ranks_and_views_agree():
    """The kernels see the same values whatever the layout, so the results are the same to the bit."""
    q, k, v = normal(2, 4, 65, 64), normal(2, 2, 65, 64, seed=1), normal(2, 2, 65, 64, seed=2)
    ref = grads(q, k, v, causal=True, softcap=8.0)
    rows = lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)                 # storage [B, S, H, D]
    part = lambda t: torch.cat([t, t], dim=-1)[..., :64]                            # rows of a wider tensor
    for view in (rows, part):
        for a, b in zip(ref, grads(view(q), view(k), view(v), causal=True, softcap=8.0)):
            assert a.shape == b.shape and torch.equal(a, b)
    for a, b in zip(ref, grads(q[:, None], k[:, None], v[:, None], causal=True, softcap=8.0)):
        assert torch.equal(a[:, None], b)


def shifted(t):
    """The same values at a base address that is 2 bytes off 16."""
    room = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    return room[1:].view(t.shape).copy_(t)


GRADIENTS = {                                        # as autograd hands them over, for an output [2, 3, 65, 64]
    "sum over the batch": lambda: normal(1, 3, 65, 64, seed=7).expand(2, 3, 65, 64),
    "mean over the heads": lambda: normal(2, 1, 65, 64, seed=8).expand(2, 3, 65, 64),
    "sum over the rows": lambda: normal(2, 3, 1, 64, seed=9).expand(2, 3, 65, 64),
    "sum over the channels": lambda: normal(2, 3, 65, 1, seed=10).expand(2, 3, 65, 64),
    "unaligned base": lambda: shifted(normal(2, 3, 65, 64, seed=11)),
    "unaligned rows": lambda: normal(2, 3, 65, 70, seed=12)[..., :64],
}


@pytest.mark.parametrize("name", list(GRADIENTS))
@pytest.mark.parametrize("entry", ["attention", "variant_attention"])
def test_output_gradients_of_any_layout(name, entry):
    """An output gradient that the kernels cannot read as it lies (broadcast or unaligned) gives what its dense copy gives."""
    x = [normal(2, 3, 65, 64, seed=n).requires_grad_(True) for n in range(3)]
    more = {} if entry == "attention" else dict(biases=[normal(1, 1, 3, 65, 65, seed=4)])
    out = getattr(F, entry)(*x, causal=True, **more)
    dout = GRADIENTS[name]()
    want = torch.autograd.grad(out, x, dout.contiguous().clone(), retain_graph=True)
    for a, b in zip(torch.autograd.grad(out, x, dout), want):
        assert torch.equal(a, b)


def test_refusals():
    q = normal(1, 2, 16, 64)
    with pytest.raises(KeyError):
        F.attention(q, q.half(), q)
    with pytest.raises(ValueError):
        F.attention(q, q, q[0])
    with pytest.raises(Exception, match="size"):
        F.attention(q, q, q[:, :, :8])
    cache = normal(4, 16, 2, 64)
    lens = torch.tensor([20], dtype=torch.int32, device="cuda:0")
    table = torch.tensor([[1, 3]], dtype=torch.int32, device="cuda:0")
    want = F.decode_attention(q[:, :, 0], cache, cache, lens, table)
    with pytest.raises(ValueError, match="workspace"):
        F.decode_attention(q[:, :, 0], cache, cache, lens, table, workspace=torch.empty(8, dtype=torch.uint8, device="cuda:0"))
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda:0")
    got, lse = F.decode_attention(q[:, :, 0], cache, cache, lens, table, workspace=ws, return_lse=True)
    assert torch.equal(got, want) and lse.shape == (1, 2) and bool(torch.isfinite(lse).all())


def variant_step(q, k, v, **kw):
    named = {n: t for n, t in kw.items() if isinstance(t, torch.Tensor)}
    x = [t.detach().requires_grad_(True) for t in (q, k, v, *named.values())]
    biases = [b.detach().requires_grad_(True) for b in kw.pop("biases", ())]
    rest = {n: t for n, t in kw.items() if n not in named}
    out = F.variant_attention(*x[:3], **dict(zip(named, x[3:])), biases=biases, **rest)
    return (out.detach(),) + torch.autograd.grad(out, x + biases, torch.ones_like(out))


@pytest.mark.parametrize("form", ["gate_bias", "two_streams", "norm_without_weight"])
def test_variant_ranks_agree(form):
    """[B, H, S, D] and [B, 1, H, S, D] reach the kernels as the same tensors, output and every gradient in its input's layout."""
    q, k, v = (normal(2, 3, 70, 64, seed=n) for n in range(3))
    if form == "gate_bias":
        kw = dict(gate=normal(2, 3, 70, 64, seed=5), biases=[normal(1, 1, 3, 70, 70, seed=6), normal(2, 1, 1, 1, 70, seed=7)])
    elif form == "two_streams":
        kw = dict(q2=normal(2, 3, 70, 64, seed=5), k2=normal(2, 3, 70, 64, seed=6), lam=torch.linspace(0.2, 0.9, 3, device="cuda:0"),
                  rms_weight=torch.linspace(0.5, 1.5, 64, device="cuda:0"), rmsnorm=True, causal=True)
    else:
        kw = dict(rmsnorm=True, gate=normal(2, 3, 70, 64, seed=5))
    five = {n: t[:, None] if isinstance(t, torch.Tensor) and t.dim() == 4 else t for n, t in kw.items()}
    for a, b in zip(variant_step(q, k, v, **dict(kw)), variant_step(q[:, None], k[:, None], v[:, None], **five)):
        assert torch.isfinite(a).all()
        assert torch.equal(a, b if a.dim() == b.dim() else b[:, 0])
    with pytest.raises(ValueError, match="expected"):
        F.variant_attention(q, k[0], v, **kw)


def test_eps_is_not_read_without_rmsnorm():
    """rms_eps=None (a caller's "no normalisation") beside rmsnorm=False."""
    q, k, v, gate = (normal(1, 2, 40, 64, seed=n) for n in range(4))
    assert torch.equal(F.variant_attention(q, k, v, gate=gate, rms_eps=None), F.variant_attention(q, k, v, gate=gate))
