"""GPU parity of the soft-cap kernels: caps from half a unit on, scores that saturate the cap in both directions, sizes around
the edges of 32- and 64-key tiles, the causal mask (partly visible tiles, rows with a single key), and values so large that
only probabilities of at most 2^8 keep the sums finite.  Oracle: fp64."""
import numpy as np
import pytest

from oracle import attention_oracle as ao
from paper_2511_02043_amd import inputs, runner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [0.5, 30.0, 41.5, 41.7])
@pytest.mark.parametrize("D,causal", [(64, False), (64, True), (128, False)])
@pytest.mark.parametrize("S,Sk,qscale", [(1, 1, 1.0), (33, 31, 1.0), (129, 65, 200.0), (200, 333, 20.0)])
def test_soft_cap(cap, D, causal, S, Sk, qscale):
    soft_cap(cap, D, causal, S, Sk, qscale)


@pytest.mark.parametrize("cap", [0.5, 30.0, 41.5, 50.0])
@pytest.mark.parametrize("S,Sk,qscale", [(1, 1, 1.0), (33, 31, 1.0), (129, 65, 200.0), (200, 333, 20.0)])
def test_soft_cap_32_key_tiles(cap, S, Sk, qscale):
    """The four-wave shape with 32-key tiles, the host's choice for key loops of up to 2048 keys on large launches."""
    from paper_2511_02043_amd import binding as fb
    try:
        fb.check(fb.fl_set_tuning("bn", 32))
        fb.check(fb.fl_set_tuning("wpe", 4))
        soft_cap(cap, 64, False, S, Sk, qscale)
    finally:
        fb.fl_set_tuning("bn", 0)
        fb.fl_set_tuning("wpe", 0)


def soft_cap(cap, D, causal, S, Sk, qscale):
    import torch
    w = inputs.causal_bf16(B=2, H=3, S=S, Sk=Sk, D=D, causal=causal, salt=21)
    w.q = inputs.round_to_bf16(w.q * np.float32(qscale))
    w.softcap = cap
    dw = runner.upload(w, out_dtype="f32")
    dw.out.fill_(float("nan"))
    dw.run_checked()
    torch.cuda.synchronize()
    ref, ref_lse = ao.run_workload(w)
    err = float(np.max(np.abs(dw.out.cpu().numpy().astype(np.float64) - ref)))
    # every probability is rounded to bf16, at most 2^-8 of itself, so the output moves by at most 2^-8 of the largest value
    # (sharp distributions come close to that: there is nothing for the rounding to average over)
    bound = 2.0 ** -8 * float(np.max(np.abs(w.v))) + 1e-4
    lse_err = float(np.max(np.abs(runner.lse_to_oracle_layout(dw) - ref_lse)))
    print(f"cap={cap} D={D} causal={causal} {S}x{Sk}: max_abs={err:.3e} lse={lse_err:.3e}", flush=True)
    assert err <= bound and lse_err <= 1e-3


@pytest.mark.parametrize("cap", [30.0, 41.7])
@pytest.mark.parametrize("D,causal,shape", [(64, False, None), (64, False, (32, 4)), (64, True, None), (128, False, None)])
def test_large_values_behind_low_scores(cap, D, causal, shape):
    """The first keys of every row score at the lower end of the cap, the later ones at the upper end, and the values are
    near 2^93: a probability may exceed the running reference by 2^8 at most, so the sums stay below 2^128."""
    import torch
    from paper_2511_02043_amd import binding as fb
    w = inputs.causal_bf16(B=1, H=2, S=200, Sk=200, D=D, causal=causal, salt=23)
    w.q[:] = 4.0
    w.k[:, :, :, :70] = -4.0
    w.k[:, :, :, 70:] = 4.0
    w.v = inputs.round_to_bf16(w.v * np.float32(2.0 ** 93))
    w.softcap = cap
    try:
        if shape is not None:
            fb.check(fb.fl_set_tuning("bn", shape[0]))
            fb.check(fb.fl_set_tuning("wpe", shape[1]))
        dw = runner.upload(w, out_dtype="f32")
        dw.out.fill_(float("nan"))
        dw.run_checked()
        torch.cuda.synchronize()
    finally:
        fb.fl_set_tuning("bn", 0)
        fb.fl_set_tuning("wpe", 0)
    ref, _ = ao.run_workload(w)
    got = dw.out.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got))
    # probabilities rounded to bf16 as above
    assert np.max(np.abs(got - ref)) <= 2.0 ** -8 * np.max(np.abs(w.v))
