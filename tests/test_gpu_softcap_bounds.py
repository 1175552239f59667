"""GPU parity of the soft-cap kernels that keep the reference of a row's first tile (caps up to 41.5) and of the general ones
beside them: caps on both sides of the line, scores that saturate the cap in both directions, sizes around the edges of
32- and 64-key tiles, the causal mask (partly visible tiles, rows with a single key).  Oracle: fp64."""
import numpy as np
import pytest

from oracle import attention_oracle as ao
from paper_2511_02043_amd import inputs, runner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [0.5, 30.0, 41.5, 41.7])
@pytest.mark.parametrize("D,causal", [(64, False), (64, True), (128, False)])
@pytest.mark.parametrize("S,Sk,qscale", [(1, 1, 1.0), (33, 31, 1.0), (129, 65, 200.0), (200, 333, 20.0)])
def test_soft_cap(cap, D, causal, S, Sk, qscale):
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
