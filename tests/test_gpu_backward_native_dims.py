"""GPU parity of the backward kernels compiled for head dim 32 and for D = 64 with Dv = 128, which read the caller's tensors
and write the caller's gradients without padded copies: sizes around the edges of their 64-row tiles and 128-row / 128-key
workgroups, grouped heads (with the group cut over several workgroups, so that partial sums of dK and dV of different widths
are added), a chunk of queries against more keys, and both gradient types (the second softmax stream adds its dV to the first
one's in fp32 before the result is rounded).  Oracle and tolerance: as for fl_attn_bwd_ex."""
import numpy as np
import pytest

from oracle import attention_backward_oracle as bo
from oracle import attention_oracle as ao
from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs, runner
from tests.test_gpu_backward_ex import REL_L2, compare

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


def bias_workload(shape):
    w = C(D=32, n_bias=1, B=2, G=2, H=4, S=100, Sk=70)
    w.biases = (inputs.normal(shape, inputs.tensor_seed(7, 9), "bf16"),)
    return w


@pytest.mark.parametrize("shape", [(1, 1, 4, 100, 70), (1, 2, 1, 1, 70), (2, 1, 4, 1, 70), (1, 1, 1, 100, 70), (2, 2, 4, 100, 70)])
def test_bias_gradient_axes(shape):
    """Bias gradients summed over every kind of axis (batch, rows, heads, queries), at sizes that no 32 x 32 block divides:
    sums of few and of many staged blocks, along the lanes of a block and across blocks."""
    compare(bias_workload(shape), "f32", label=f"bias_{shape}")


@pytest.mark.parametrize("S", [1, 5, 31, 32])
@pytest.mark.parametrize("variant", [dict(D=32), dict(D=64), dict(D=64, pos_mask="prefix")], ids=["d32", "d64", "d64_prefix"])
def test_bias_gradients_of_few_query_rows(S, variant):
    """Staged blocks of as many rows as the call has: a bias per query and key, and one that is summed over the queries; under a
    mask (every row sees the 45 keys of the prefix) with the blocks cleared first."""
    w = C(S=S, Sk=70, n_bias=2, G=2, **variant)
    dout = inputs.dout_for(w)
    db = runner.upload_backward_ex(w, dout, grad_dtype="f32")
    db.fwd.run_checked()
    for t in db.grads["dbias"]:
        t.fill_(float("nan"))
    db.run_checked()
    for t, r in zip(db.grads["dbias"], bo.variant_backward(w, dout)["dbias"]):
        # relative L2 as for fl_attn_bwd_ex; no bound per element, since the rounding of one row's few terms does not average
        # out (see above)
        got = t.cpu().numpy().astype(np.float64)
        rel = float(np.sqrt(np.sum((got - r) ** 2) / np.sum(r * r)))
        print(f"bias2_{S}x70: rel_l2={rel:.3e}", flush=True)
        assert got.shape == r.shape and rel <= REL_L2


@pytest.mark.parametrize("shape", [(2, 2, 4, 1, 1), (1, 1, 4, 100, 1), (1, 1, 1, 1, 1)])
def test_bias_gradient_summed_over_the_keys(shape):
    """A bias that is the same for all keys of a row does not change the softmax: its gradient is zero in real arithmetic.  What
    may be left is the rounding of dS to bf16 and that of the stored output, which enters delta = rowsum(dout * out): 2^-9 of
    each term (2^-8 allowed, for the fp32 arithmetic before it)."""
    w = bias_workload(shape)
    dout = inputs.dout_for(w)
    db = runner.upload_backward_ex(w, dout, grad_dtype="f32")
    db.fwd.run_checked()
    for t in db.grads["dbias"]:
        t.fill_(float("nan"))
    db.run_checked()
    got = db.grads["dbias"][0].cpu().numpy().astype(np.float64)
    out, _ = ao.run_workload(w)
    w.biases = (np.ascontiguousarray(np.broadcast_to(w.biases[0], (2, 2, 4, 100, 70))),)
    ds = bo.variant_backward(w, dout)["dbias"][0]
    terms = np.abs(ds).sum(-1, keepdims=True) + np.abs(dout.astype(np.float64) * out).sum(-1, keepdims=True)
    bound = 2.0 ** -8 * terms.sum(tuple(a for a in range(4) if shape[a] == 1), keepdims=True)
    assert got.shape == shape
    assert np.all(np.abs(got) <= bound), (float(np.max(np.abs(got))), float(np.max(bound)))
