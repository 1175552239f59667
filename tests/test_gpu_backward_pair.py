"""The stationary-bias backward kernels (a pair bias shared by the row problems, with or without a key bias): dQ, dK, dV and both
bias gradients against the fp64 oracle where tiles end -- 32-row blocks, 64 owned rows, steps of 128 streamed rows, ranges of the
row axis -- and against the general kernels, which take the same calls with the tuning switch.  Tolerance: fl_attn_bwd_ex's
(P and dS in bf16, fp32 sums; relative L2 <= 5e-3)."""
import numpy as np
import pytest
import torch

from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs, runner
from test_gpu_backward_ex import compare

pytestmark = pytest.mark.gpu

C = inputs.combination_bf16


@pytest.mark.parametrize("n_bias", [1, 2])
@pytest.mark.parametrize("D,Sq,Sk,G,H", [(32, 1, 1, 2, 1), (32, 31, 33, 3, 2), (32, 64, 128, 9, 1), (32, 65, 129, 2, 2), (32, 257, 200, 3, 1), (32, 384, 300, 2, 2),
                                         (32, 385, 511, 2, 1), (32, 512, 40, 2, 1), (64, 33, 64, 5, 2), (64, 128, 65, 2, 2), (64, 129, 256, 3, 1), (64, 300, 384, 2, 1)])
def test_sizes(D, Sq, Sk, G, H, n_bias):
    compare(C(D=D, n_bias=n_bias, S=Sq, Sk=Sk, G=G, B=2, H=H), "f32", label=f"D {D} {Sq} x {Sk} G {G} H {H} biases {n_bias}")


def _grads(w, dout, tune, grad_dtype="f32"):
    fb.check(fb.fl_set_tuning("pair_bias", tune))
    try:
        db = runner.upload_backward_ex(w, dout, grad_dtype=grad_dtype)
        db.fwd.run_checked()
        out = []
        for _ in range(2):
            for t in db.grads.values():
                for x in (t if isinstance(t, list) else [t]):
                    x.fill_(float("nan"))
            db.run_checked()
            torch.cuda.synchronize()
            out.append({f"{n}{i}": x.float().cpu().numpy().copy() for n, t in db.grads.items()
                        for i, x in enumerate(t if isinstance(t, list) else [t])})
    finally:
        fb.fl_set_tuning("pair_bias", 0)
    for n in out[0]:
        assert np.array_equal(out[0][n], out[1][n], equal_nan=True), f"{n} differs between two runs"
    return out[0]


# key bias first, pair bias shared by the batch too, bf16 gradients, as few row problems as there can be; odd bias rows throughout
@pytest.mark.parametrize("form", ["plain", "key_first", "pair_over_batch", "bf16", "one_range"])
@pytest.mark.parametrize("D", [32, 64])
def test_same_as_general_kernels(D, form):
    G = 2 if form == "one_range" else 20
    w = inputs.evoformer_bf16(B=2, Nseq=G, Nres=203, H=2, D=D, two_biases=True, salt=5)
    pair, key = w.biases
    if form == "key_first":
        w.biases = (key, pair)
    elif form == "pair_over_batch":
        w.biases = (pair[:1], key)
    dout = inputs.dout_for(w)
    dtype = "bf16" if form == "bf16" else "f32"
    new, old = _grads(w, dout, 0, dtype), _grads(w, dout, 1, dtype)
    assert new.keys() == old.keys() and any(n.startswith("dbias") for n in new)
    for n in new:
        assert np.all(np.isfinite(new[n])), n
        rel = np.linalg.norm(new[n] - old[n]) / np.linalg.norm(old[n])
        print(f"{form} D {D} {n}: {rel:.2e}", flush=True)
        assert rel <= 4e-3, n                      # both round P and dS to bf16 (2^-9 each), from differently rounded exponents
    assert not all(np.array_equal(new[n], old[n]) for n in new), "the switch chose the same kernels"


@pytest.mark.parametrize("hide", [-np.inf, -1e9])
def test_hidden_keys(hide):
    """A key bias that hides keys: their gradients are zero, and so are those of a row problem without any visible key under
    -inf (lse = -inf)."""
    w = inputs.evoformer_bf16(B=1, Nseq=6, Nres=150, H=2, D=32, two_biases=True, salt=9)
    key = w.biases[1].copy()
    key[0, 0, 0, 0, 100:] = hide
    key[0, 2, 0, 0, :70] = hide
    if np.isinf(hide):
        key[0, 4] = hide
    w.biases = (w.biases[0], inputs.round_to_bf16(key))
    g = _grads(w, inputs.dout_for(w), 0)
    for n, x in g.items():
        assert np.all(np.isfinite(x)), n
    assert np.all(g["dk0"][0, 0, :, 100:] == 0) and np.all(g["dv0"][0, 0, :, 100:] == 0) and np.all(g["dk0"][0, 2, :, :70] == 0)
    assert np.any(g["dk0"][0, 0, :, :100] != 0) and np.any(g["dk0"][0, 2, :, 70:] != 0)
    if np.isinf(hide):
        assert all(np.all(g[n][0, 4] == 0) for n in ("dq0", "dk0", "dv0"))
    old = _grads(w, inputs.dout_for(w), 1)
    for n in g:
        assert np.linalg.norm(g[n] - old[n]) <= 4e-3 * np.linalg.norm(old[n]), n
