"""fp32 storage: the workgroup shapes (row groups x key splits) of the fp32 kernel at the edges of their ranges, head dims
below the kernels' own, and every variant feature with several key splits; against the fp64 oracle."""
import numpy as np
import pytest

from paper_2511_02043_amd import inputs
from tests.gpu_util import run_and_compare

pytestmark = pytest.mark.gpu


def as_f32(w):
    w.dtype = "f32"
    w.name += "_as_f32"
    return w


def differential_128():
    w = inputs.combination_bf16(D=128, Dv=128, diff=True, rmsnorm=True, gate=True, pos_mask="causal", n_bias=2, B=1, S=130)
    return as_f32(w)


# B, H, S, Sk, D: launches that take 1, 2, 4 and 8 key splits at each head dim, ragged against the 32-row groups and 32-key
# tiles; key counts below the number of splits' tiles
@pytest.mark.parametrize("B,H,S,Sk,D", [
    (8, 32, 40, 33, 32), (4, 33, 129, 65, 32), (2, 40, 97, 200, 32), (1, 2, 33, 300, 32), (1, 1, 1, 31, 20),
    (8, 32, 33, 97, 64), (4, 32, 130, 40, 64), (1, 3, 65, 161, 64), (1, 2, 31, 1, 36), (1, 2, 64, 257, 60),
    (8, 32, 31, 64, 128), (4, 32, 129, 33, 128), (1, 2, 70, 225, 128), (1, 3, 1, 129, 100), (2, 2, 33, 32, 68),
])
def test_f32_workgroup_shapes(B, H, S, Sk, D):
    run_and_compare(inputs.plain_f32(B=B, H=H, S=S, Sk=Sk, D=D))


@pytest.mark.parametrize("make", [
    lambda: as_f32(inputs.causal_bf16(B=1, H=4, S=333, D=128, Hkv=2)),
    lambda: as_f32(inputs.causal_bf16(B=8, H=32, S=257, D=32)),                 # one key split, two row tiles
    lambda: as_f32(inputs.combination_bf16(D=32, Dv=128, score_mod="softcap", pos_mask="window", doc=True, n_bias=2, S=201)),
    lambda: as_f32(inputs.combination_bf16(D=128, Dv=32, score_mod="alibi", pos_mask="prefix", doc=True, gate=True, S=170, Sk=140)),
    lambda: as_f32(inputs.combination_bf16(D=64, Dv=128, diff=True, rmsnorm=True, doc=True, pos_mask="causal", S=140)),
    differential_128,
], ids=["causal_gqa_d128", "causal_d32_many", "window_doc_bias_d32_128", "prefix_doc_gate_d128_32", "diff_rms_doc", "diff_rms_gate_d128"])
def test_f32_variants_over_key_splits(make):
    run_and_compare(make())
