"""The dK/dV kernel with 64 keys per wave against the fp64 oracle where its tiles end: 32-row blocks, 64-row tiles (rings of three), 64 keys
of a wave, 256 of a workgroup; every variant that has one, grouped heads in one piece and cut.  The tuning switch selects it for calls of any
size.  Tolerance: fl_attn_bwd's (P and dS in bf16, fp32 sums; relative L2 <= 5e-3)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import attention_backward_oracle as bo
from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs, runner
import test_gpu_backward as simple

pytestmark = pytest.mark.gpu


@pytest.fixture
def always():
    fb.check(fb.fl_set_tuning("bwd_keys", 2))
    yield
    fb.fl_set_tuning("bwd_keys", 0)


SIZES = [(1, 1), (31, 63), (65, 64), (200, 255), (129, 257), (320, 256), (333, 600)]
VARIANTS = {
    "plain": lambda **k: inputs.causal_bf16(causal=False, **k),
    "causal": lambda **k: inputs.causal_bf16(**k),
    "alibi": lambda **k: dataclasses.replace(inputs.causal_bf16(causal=False, **k), alibi=np.array([0.25, 0.01], np.float32)),
    "softcap": lambda **k: dataclasses.replace(inputs.causal_bf16(causal=False, **k), softcap=2.0),
    "prefix": lambda **k: dataclasses.replace(inputs.causal_bf16(causal=False, **k), prefix=70),
}


@pytest.mark.parametrize("Sq,Sk", SIZES)
@pytest.mark.parametrize("variant", list(VARIANTS))
def test_sizes(variant, Sq, Sk, always):
    simple.compare(VARIANTS[variant](B=1, H=2, S=Sq, Sk=Sk, D=128), label=f"{variant} {Sq} x {Sk}")


@pytest.mark.parametrize("wgs", [0, 4096])
def test_grouped_heads(wgs, always):
    fb.check(fb.fl_set_tuning("bwd_wg_target", wgs))
    try:
        simple.compare(inputs.causal_bf16(B=2, H=8, Hkv=2, S=391, D=128), "bf16", label="grouped")
    finally:
        fb.fl_set_tuning("bwd_wg_target", 0)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("S", [33, 65, 257, 400])
def test_differential(S, causal, always):
    """What the kernel makes of the two streams: dK, dK2 and dV, which the second stream's pass adds to the first one's."""
    w = inputs.differential_bf16(B=1, H=2, S=S, D=64, Dv=128, causal=causal, rmsnorm=False)
    dout = inputs.dout_for(w)
    db = runner.upload_backward_ex(w, dout, grad_dtype="f32")
    db.fwd.run_checked()
    db.run_checked()
    torch.cuda.synchronize()
    ref = bo.variant_backward(w, dout)
    for name in ("dk", "dk2", "dv"):
        diff = db.grads[name].cpu().numpy() - ref[name]
        assert np.sqrt(np.sum(diff * diff) / np.sum(ref[name] ** 2)) <= simple.REL_L2, name


def test_same_as_128_keys_and_reproducible():
    """The sums of a key run over the rows in the same order: up to dS's last bit before its rounding, the results are the same."""
    w = inputs.causal_bf16(B=64, H=8, S=255, D=128)          # taken by the host's rule
    dout = inputs.dout_for(w)
    db = runner.upload_backward(w, dout, grad_dtype="f32")
    db.fwd.run_checked()
    got = []
    for keys in (0, 0, 2, 1):
        fb.check(fb.fl_set_tuning("bwd_keys", keys))
        try:
            for t in (db.dk, db.dv):
                t.fill_(float("nan"))
            db.run_checked()
            torch.cuda.synchronize()
        finally:
            fb.fl_set_tuning("bwd_keys", 0)
        got.append([t.cpu().numpy() for t in (db.dk, db.dv)])
    for n in range(2):
        assert np.array_equal(got[0][n], got[1][n]) and np.array_equal(got[0][n], got[2][n])
        diff = got[0][n] - got[3][n]
        assert np.sqrt(np.sum(diff * diff) / np.sum(got[3][n] ** 2)) < 1e-3
    assert not np.array_equal(got[0][0], got[3][0])          # two kernels, not one


@pytest.mark.parametrize("variant,B,H,Hkv,S,wide", [
    ("causal", 18, 16, 16, 289, False), ("causal", 6, 16, 16, 1641, True), ("causal", 2, 16, 2, 807, False), ("prefix", 5, 16, 16, 1490, True),
    ("plain", 7, 32, 32, 370, False), ("plain", 8, 16, 16, 977, True), ("alibi", 2, 8, 8, 588, False), ("alibi", 5, 32, 32, 241, True),
    ("softcap", 6, 16, 16, 843, False), ("softcap", 3, 16, 16, 800, True), ("softcap", 64, 8, 8, 351, False)])
def test_kernel_of_a_call(variant, B, H, Hkv, S, wide):
    """The faster kernel of the two, as measured for these calls; the last bits of dK tell which one ran."""
    gen = torch.Generator(device="cuda:0").manual_seed(S)
    q, k, v, dout = (torch.randn(B, 1, h, S, 128, generator=gen, device="cuda:0").to(torch.bfloat16) for h in (H, Hkv, Hkv, H))
    desc = fb.variant_desc(scale=128 ** -0.5, mask={"causal": fb.FL_MASK_CAUSAL, "prefix": fb.FL_MASK_PREFIX}.get(variant, 0), prefix_len=256 if variant == "prefix" else 0,
                           score_mod={"alibi": fb.FL_MOD_ALIBI, "softcap": fb.FL_MOD_SOFTCAP}.get(variant, 0), softcap=30.0 if variant == "softcap" else 0.0)
    slopes = torch.linspace(0.01, 0.5, H, device="cuda:0") if variant == "alibi" else None
    got = [gradients(keys, q, k, v, dout, desc, slopes)[0] for keys in (0, 1, 2)]
    assert not torch.equal(got[1], got[2])
    assert torch.equal(got[0], got[2 if wide else 1])


@pytest.mark.parametrize("Sq,Sk,off", [(130, 700, 570), (130, 700, 150), (333, 600, 1), (64, 257, 193), (1, 300, 299)])
@pytest.mark.parametrize("variant", ["causal", "prefix", "alibi"])
def test_rows_at_an_offset(variant, Sq, Sk, off, always):
    """A chunk of rows against more keys; keys behind the chunk, which no row sees, get exactly zero."""
    w = VARIANTS[variant](B=1, H=2, S=Sq, Sk=Sk, D=128)
    w.q_offset = off
    simple.compare(w, label=f"{variant} {Sq} of {Sk} at {off}")
    if variant != "alibi":
        _, (_, dk, dv) = simple.run_backward(w)
        unseen = max(off + Sq, 70 if variant == "prefix" else 0)
        assert np.all(dk[..., unseen:, :] == 0) and np.all(dv[..., unseen:, :] == 0)


def gradients(keys, q, k, v, dout, desc, slopes=None, spoil=None):
    """dK and dV of tensors with any strides on the kernel that `keys` asks for; spoil(lse): what is done to the forward pass's lse."""
    out, lse = torch.empty_like(q), torch.empty(*q.shape[:4], 1, device="cuda:0")
    grads = [torch.full(x.shape, float("nan"), device="cuda:0") for x in (q, k, v)]
    t = [fb.tensor_desc(x) for x in (q, k, v, out, dout, lse, *grads)]
    need = max(fb.fl_attn_fwd_workspace_size(t[0], t[1], desc), fb.fl_attn_bwd_workspace_size(t[0], t[1], desc), 16)
    aux = fb.aux_desc(alibi_slopes=slopes, workspace=torch.empty(need, dtype=torch.uint8, device="cuda:0"))
    stream = torch.cuda.current_stream().cuda_stream
    fb.check(fb.fl_attn_fwd(t[0], t[1], t[2], desc, aux, t[3], t[5], stream))
    if spoil is not None:
        spoil(lse)
    fb.check(fb.fl_set_tuning("bwd_keys", keys))
    try:
        fb.check(fb.fl_attn_bwd(*t[:6], desc, aux, *t[6:], stream))
        torch.cuda.synchronize()
    finally:
        fb.fl_set_tuning("bwd_keys", 0)
    return grads[1:]


def normal(*shape, seed=0):
    return torch.randn(shape, generator=torch.Generator(device="cuda:0").manual_seed(seed), device="cuda:0").to(torch.bfloat16)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,G,H,Hkv,Sq,Sk", [(2, 1, 4, 2, 333, 300), (1, 3, 2, 2, 130, 257), (2, 2, 4, 4, 65, 600)])
def test_strides_and_row_axes(B, G, H, Hkv, Sq, Sk, causal):
    """Heads side by side in storage, rows of a wider buffer, several problems along G: the bits of dense tensors."""
    desc = fb.variant_desc(scale=128 ** -0.5, mask=fb.FL_MASK_CAUSAL if causal else 0)
    view = lambda h, s, wide, seed: normal(B, G, s, h, wide, seed=seed)[..., wide - 128:].transpose(2, 3)     # [B, G, h, s, 128]
    q, k, v, dout = view(H, Sq, 256, 1), view(Hkv, Sk, 128, 2), view(Hkv, Sk, 192, 3), view(H, Sq, 136, 4)
    assert not q.is_contiguous() and dout.stride(3) == H * 136
    strided = gradients(2, q, k, v, dout, desc)
    dense = gradients(2, *(x.contiguous() for x in (q, k, v, dout)), desc)
    other = gradients(1, q, k, v, dout, desc)
    for a, b, c in zip(strided, dense, other):
        assert torch.equal(a, b) and float((a - c).norm() / c.norm()) < 1e-3


@pytest.mark.parametrize("variant", ["plain", "causal", "softcap"])
@pytest.mark.parametrize("row", [5, 100, 198])
def test_a_row_whose_lse_is_nan(variant, row):
    """Its keys get NaN and no others do, with 64 and 32 keys per wave: rows inside a tile and the last one, which stands in for rows past the end."""
    Sq, Sk, off = 199, 400, 30
    q, k, v, dout = normal(1, 1, 2, Sq, 128, seed=5), normal(1, 1, 2, Sk, 128, seed=6), normal(1, 1, 2, Sk, 128, seed=7), normal(1, 1, 2, Sq, 128, seed=8)
    desc = fb.variant_desc(scale=128 ** -0.5, mask=fb.FL_MASK_CAUSAL if variant == "causal" else 0, q_offset=off if variant == "causal" else 0,
                           score_mod=fb.FL_MOD_SOFTCAP if variant == "softcap" else 0, softcap=30.0 if variant == "softcap" else 0.0)

    def spoil(lse):
        lse[0, 0, 0, row] = float("nan")
    wide, narrow = (gradients(keys, q, k, v, dout, desc, spoil=spoil) for keys in (2, 1))
    seen = row + off + 1 if variant == "causal" else Sk
    for a, b in zip(wide, narrow):
        assert a[0, 0, 0, :seen].isnan().all() and not a[0, 0, 0, seen:].isnan().any() and not a[0, 0, 1].isnan().any()
        assert torch.equal(a.isnan(), b.isnan())
        assert float((a - b)[~a.isnan()].norm() / b[~b.isnan()].norm()) < 1e-3
