"""GPU parity of the backward kernels compiled for head dim 32 and for D = 64 with Dv = 128, which read the caller's tensors
and write the caller's gradients without padded copies: sizes around the edges of their 64-row tiles and 128-row / 128-key
workgroups, grouped heads (with the group cut over several workgroups, so that partial sums of dK and dV of different widths
are added), a chunk of queries against more keys, and both gradient types (the second softmax stream adds its dV to the first
one's in fp32 before the result is rounded).  Oracle and tolerance: as for fl_attn_bwd_ex."""
import pytest

from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs
from tests.test_gpu_backward_ex import compare

pytestmark = pytest.mark.gpu

C = inputs.combination_bf16
VARIANTS = {
    "plain_d32": dict(D=32),
    "causal_d32_gqa": dict(D=32, pos_mask="causal", H=4, Hkv=1),
    "bias1_gate_d32": dict(D=32, n_bias=1, gate=True),
    "bias2_d32": dict(D=32, n_bias=2, G=2, B=1),
    "d64_dv128_gqa": dict(D=64, Dv=128, H=4, Hkv=2),
    "diff_rms_causal_d64_dv128": dict(D=64, Dv=128, pos_mask="causal", diff=True, rmsnorm=True, H=4, Hkv=2),
}


# (At least 33 keys: the tolerance assumes that rounding averages out over a row.  With three, a row's largest probability p
# is close to 1, dS = p (dP - delta) is what is left of a cancellation by 1 - p, and delta carries the 2^-9 by which each
# channel of the stored output is rounded: 2^-9 / (1 - p) relative, over 1e-2 for p above 0.8.)
@pytest.mark.parametrize("S,Sk", [(33, 33), (31, 65), (64, 64), (129, 127), (200, 333)])
@pytest.mark.parametrize("name", list(VARIANTS))
def test_sizes(name, S, Sk):
    compare(C(S=S, Sk=Sk, **VARIANTS[name]), "f32", label=f"{name}_{S}x{Sk}")


@pytest.mark.parametrize("name", ["causal_d32_gqa", "diff_rms_causal_d64_dv128"])
def test_bf16_gradients_and_split_groups(name):
    fb.check(fb.fl_set_tuning("bwd_wg_target", 1 << 20))      # cut every group as far as it goes
    try:
        compare(C(S=150, Sk=150, **VARIANTS[name]), "bf16", label=name)
        compare(C(S=150, Sk=150, **VARIANTS[name]), "f32", label=name)
    finally:
        fb.fl_set_tuning("bwd_wg_target", 0)
