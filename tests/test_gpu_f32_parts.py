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
