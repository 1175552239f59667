"""fp32 storage: the workgroup shapes (row groups x key splits) of the fp32 kernel at the edges of their ranges, head dims
below the kernels' own, and every variant feature with several key splits; against the fp64 oracle."""
import dataclasses

import numpy as np
import pytest

from oracle import attention_oracle as ao
from paper_2511_02043_amd import inputs, runner
from tests.gpu_util import TOL, run_and_compare

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


def run_f32(w):
    import torch
    dw = runner.upload(w)
    dw.out.fill_(float("nan"))
    dw.run_checked()
    torch.cuda.synchronize()
    return dw.out.cpu().numpy().astype(np.float64), runner.lse_to_oracle_layout(dw)


# launches of 8, 2 and 1 row groups (see above)
SHAPES = [(8, 32, 33, 20), (8, 32, 33, 36), (8, 32, 33, 100), (2, 40, 97, 20), (1, 3, 65, 60), (1, 2, 33, 28), (1, 2, 70, 124)]


@pytest.mark.parametrize("B,H,S,D", SHAPES)
def test_f32_infinite_key_at_a_head_dim_below_the_kernels(B, H, S, D):
    """A key whose first channel is infinite scores -inf and has no weight; the channels that the kernel adds past D must not
    turn it into a NaN."""
    w = inputs.plain_f32(B=B, H=H, S=S, Sk=70, D=D)
    w.q[..., 0] = np.abs(w.q[..., 0]) + 0.5
    for j in (3, 40, 69):
        w.k[:, :, :, j, 0] = -np.inf
    got, lse = run_f32(w)
    keep = np.isfinite(w.k[0, 0, 0, :, 0])
    sub = dataclasses.replace(w, k=w.k[:, :, :, keep], v=w.v[:, :, :, keep])
    ref, ref_lse = ao.run_workload(sub)
    assert np.max(np.abs(got - ref)) <= TOL["f32"]["max_abs"] and np.max(np.abs(lse - ref_lse)) <= TOL["f32"]["lse"]


@pytest.mark.parametrize("B,H,S,D", SHAPES + [(8, 32, 33, 64), (1, 2, 64, 128), (1, 1, 31, 32)])
def test_f32_infinite_value_of_the_last_key(B, H, S, D):
    """70 keys end inside a tile: the rows that fill it up are copies of the last key and have to count for nothing, also where
    its value is infinite."""
    w = inputs.plain_f32(B=B, H=H, S=S, Sk=70, D=D)
    ref, _ = ao.run_workload(w)
    w.v[:, :, :, 69, 5] = np.inf
    got, _ = run_f32(w)
    assert np.all(np.isposinf(got[..., 5]))
    rest = np.arange(D) != 5
    assert np.max(np.abs(got[..., rest] - ref[..., rest])) <= TOL["f32"]["max_abs"]
