"""fp32 storage without score_mod, biases or epilogue: contractions on three bf16 parts of each operand, and the pass on the fp32
matrix instruction that takes over where the parts cannot hold a value; against the fp64 oracle."""
import numpy as np
import pytest

from oracle import attention_oracle as ao
from paper_2511_02043_amd import inputs, runner

pytestmark = pytest.mark.gpu

# Relative L2 error: operands are held to 2^-24 (their own rounding), products to 2^-26, sums are fp32: a few 1e-7 (measured up to 8e-7)
REL = 2e-6


def run(w):
    import torch
    dw = runner.upload(w)
    dw.out.fill_(float("nan"))
    dw.run_checked()
    torch.cuda.synchronize()
    return dw.out.cpu().numpy().astype(np.float64), runner.lse_to_oracle_layout(dw)


def compare(w):
    got, lse = run(w)
    ref, ref_lse = ao.run_workload(w)
    assert np.sqrt(np.sum((got - ref) ** 2)) <= REL * np.sqrt(np.sum(ref ** 2)), w.name
    assert np.max(np.abs(lse - ref_lse)) <= 1e-5, w.name


# B, H, S, Sk, D: one and two row blocks per wave, every number of key splits at each head dim, ragged against 32, 64, 128, 256 and
# 512 rows and 32 keys, head dims below the kernels' own
@pytest.mark.parametrize("B,H,S,Sk,D", [
    (4, 32, 1025, 65, 32), (4, 32, 511, 33, 32), (2, 40, 513, 300, 20), (2, 32, 255, 97, 32), (1, 2, 65, 31, 32),
    (4, 32, 1025, 40, 64), (4, 32, 257, 65, 64), (2, 32, 449, 161, 60), (2, 32, 255, 257, 64), (1, 2, 63, 1, 64),
    (4, 32, 257, 64, 128), (2, 33, 500, 95, 100), (2, 33, 255, 225, 128), (1, 2, 33, 129, 128),
])
def test_shapes(B, H, S, Sk, D):
    compare(inputs.plain_f32(B=B, H=H, S=S, Sk=Sk, D=D))


@pytest.mark.parametrize("B,H,S,Sk,D", [(64, 8, 64, 64, 64), (64, 8, 32, 32, 64), (64, 8, 33, 100, 64), (64, 8, 100, 129, 60), (64, 8, 64, 33, 32),
                                        (64, 8, 1, 300, 64), (64, 8, 17, 256, 32), (32, 8, 513, 65, 64), (32, 8, 257, 97, 20)])
def test_many_problems_of_few_rows(B, H, S, Sk, D):
    """Workgroups of fewer rows although the launch fills the chip without; one tile of keys and up to ten, ends of the row and key tiles."""
    compare(inputs.plain_f32(B=B, H=H, S=S, Sk=Sk, D=D))


@pytest.mark.parametrize("B,H,S,D", [(2, 8, 300, 32), (2, 8, 300, 64), (2, 8, 300, 128), (4, 32, 257, 64), (4, 32, 257, 128)])
@pytest.mark.parametrize("q,k,v", [(1, 1, 2.0 ** -118), (2.0 ** -112, 2.0 ** 112, 1), (2.0 ** 112, 2.0 ** -112, 1), (1, 1, 2.0 ** 122), (1, 1, 0)])
def test_magnitudes(B, H, S, D, q, k, v):
    """The third part of a value below 2^-110 or so is below what bf16 holds; the result has to be as good as anywhere else.  A power of two
    in the scores is taken out again by its inverse, so that the oracle's are those of the plain case."""
    w = inputs.plain_f32(B=B, H=H, S=S, Sk=200, D=D)
    w.q, w.k, w.v = (x * np.float32(f) for x, f in ((w.q, q), (w.k, k), (w.v, v)))
    compare(w)


@pytest.mark.parametrize("D", [32, 64, 128])
def test_single_values_outside(D):
    """A column of tiny values and one value that rounds to a bf16 infinity, among ordinary ones: each column keeps its precision."""
    w = inputs.plain_f32(B=2, H=8, S=300, Sk=200, D=D)
    w.v[..., 3] *= np.float32(2.0 ** -118)
    w.v[:, :, :, 7, 5] = np.float32(3.4e38)
    got, _ = run(w)
    ref, _ = ao.run_workload(w)
    for c in range(D):
        size = np.max(np.abs(ref[..., c]))
        assert np.sqrt(np.sum(((got[..., c] - ref[..., c]) / size) ** 2)) <= REL * np.sqrt(np.sum((ref[..., c] / size) ** 2)), c


# B, H, S: workgroups of one row group (waves that decide alone) and of several (waves that share tiles)
BOTH = [(2, 8, 300), (4, 32, 257)]


@pytest.mark.parametrize("B,H,S", BOTH)
@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("q,k,scale", [(0, -116, 116), (0, -120, 120), (60, -120, 60), (-60, -60, 120), (0, 30, -30), (90, -60, -30)])
def test_scales(B, H, S, D, q, k, scale):
    """Powers of two in q, k and the scale that take each other out: what the parts of k lose, the scale must not bring back."""
    w = inputs.plain_f32(B=B, H=H, S=S, Sk=200, D=D)
    w.q, w.k = w.q * np.float32(2.0 ** q), w.k * np.float32(2.0 ** k)
    w.scale *= 2.0 ** scale
    compare(w)


@pytest.mark.parametrize("B,H,S", BOTH)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_large_values_of_small_weight(B, H, S, D):
    """Weights of 2^-123, of which bf16 parts hold ten bits, beside values of 2^126: most of the result, and of ordinary size.  The
    scores are single products of fp32 values; in the exponent, 2^-18 from the product with log2(e) and as much from its factor
    (2^-25 of 123), times ln 2."""
    w = inputs.plain_f32(B=B, H=H, S=S, Sk=200, D=D)
    w.scale = 0.125
    w.q[...], w.k[...] = 0, 0
    w.q[..., 0] = 8
    w.k[:, :, :, 20:180:16, 0] = np.float32(-85.2) + np.float32(0.03) * np.arange(10, dtype=np.float32)
    w.v[:, :, :, 20:180:16] = np.abs(w.v[:, :, :, 20:180:16]).clip(0.25, 1.9) * np.float32(2.0 ** 126)
    got, _ = run(w)
    ref, _ = ao.run_workload(w)
    assert 0.1 < np.median(np.abs(ref)) < 1e3
    assert np.sqrt(np.sum((got - ref) ** 2)) <= 1e-5 * np.sqrt(np.sum(ref ** 2))


@pytest.mark.parametrize("B,H,S", BOTH)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_values_near_the_smallest(B, H, S, D):
    """Values of 2^-136, zero in every bf16 part.  Sums and results are multiples of 2^-149: each of 2000 additions may take half of that from a
    sum of 2^-133 (the weights of a row add up to 2^4 and more, the values are 2^-137 and more), the division from a result of 2^-137."""
    w = inputs.plain_f32(B=B, H=H, S=S, Sk=2000, D=D)
    w.v = np.abs(w.v).clip(0.5, 2).astype(np.float32) * np.float32(2.0 ** -136)
    got, _ = run(w)
    ref, _ = ao.run_workload(w)
    assert np.max(np.abs(got / ref - 1)) <= 2000 * 2.0 ** -17 + 2.0 ** -13


def variant(part, D, B, H, S):
    w = inputs.combination_bf16(D=D, B=B, H=H, S=S, **part)
    w.dtype = "f32"
    return w


# every feature that only the kernels with switches have, and the masks of those without
PARTS = [dict(pos_mask="causal"), dict(pos_mask="window"), dict(pos_mask="prefix", doc=True), dict(score_mod="softcap", n_bias=2),
         dict(score_mod="alibi", pos_mask="causal", gate=True), dict(diff=True, pos_mask="causal"), dict(diff=True, rmsnorm=True, gate=True)]


WHERE = [(part, where) for part in PARTS for where in ("q", "q2", "row", "v")
         if not (where == "q2" and "diff" not in part) and not (where == "v" and "rmsnorm" in part)]


@pytest.mark.parametrize("B,H,S", BOTH)
@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("part,where", WHERE, ids=str)
def test_second_pass_of_variants(B, H, S, D, part, where):
    """What the parts cannot hold, in calls with masks, biases and a second stream: all of q (taken out again in k), of the second
    stream's only, one row's (one wave's of a workgroup), or all values (not before an RMSNorm, whose epsilon they would meet)."""
    w = variant(part, D, B, H, S)
    up, down = np.float32(2.0 ** 112), np.float32(2.0 ** -112)
    if where == "q":
        w.q, w.k = w.q * up, w.k * down
    elif where == "q2":
        w.q2, w.k2 = w.q2 * up, w.k2 * down
    elif where == "row":
        w.q = w.q.copy()
        w.q[:, :, :, 40, 1] = np.float32(2.0 ** -112)
    else:
        w.v = w.v * np.float32(2.0 ** -118)
    got, lse = run(w)
    ref, ref_lse = ao.run_workload(w)
    dead = np.isneginf(ref_lse)
    assert np.array_equal(np.isneginf(lse), dead) and np.max(np.abs(lse[~dead] - ref_lse[~dead])) <= 1e-5
    # (the difference of two streams is smaller than either)
    assert np.sqrt(np.sum((got - ref) ** 2)) <= (4 if w.q2 is not None else 1) * REL * np.sqrt(np.sum(ref ** 2))
