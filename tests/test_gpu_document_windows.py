"""Document masks over tile lists longer than the 64 tiles whose id ranges a workgroup holds at a time: documents whose tokens
recur a whole such window later (nothing visible in between), rows that see nothing in the first window, and in the dK/dV
kernels a workgroup that walks several query heads and returns to the first window for each.  Oracle: fp64."""
import numpy as np
import pytest

from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs
from tests.gpu_util import run_and_compare
from tests.test_gpu_backward import compare

pytestmark = pytest.mark.gpu

S = 4700                                             # 74 tiles of 64, 147 of 32


def recurring(D, mask, H=2, Hkv=1):
    """Document 0 at both ends, document 1 over the 4350 tokens between, document 2 at the very end."""
    w = inputs.combination_bf16(D=D, pos_mask=mask, B=1, H=H, Hkv=Hkv, S=S, window=4650, prefix=100)
    ids = np.repeat(np.array([0, 1, 0, 2], np.int32), [150, 4350, 100, 100])[None]
    w.q_doc = w.kv_doc = ids
    return w


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("mask", ["none", "causal", "window", "prefix"])
def test_forward(D, mask):
    run_and_compare(recurring(D, mask), label=f"recurring documents {mask} D={D}")


def test_forward_of_32_key_tiles():
    try:
        fb.check(fb.fl_set_tuning("bn", 32))
        fb.check(fb.fl_set_tuning("wpe", 3))
        for mask in ("none", "causal", "window"):
            run_and_compare(recurring(64, mask), label=f"recurring documents {mask} D=64, 32-key tiles")
    finally:
        fb.fl_set_tuning("bn", 0)
        fb.fl_set_tuning("wpe", 0)


@pytest.mark.parametrize("D,mask", [(64, "none"), (64, "causal"), (64, "window"), (128, "causal"), (128, "window")])
def test_backward(D, mask):
    fb.check(fb.fl_set_tuning("bwd_wg_target", 1))   # no group is cut: a workgroup walks both heads
    try:
        compare(recurring(D, mask), label=f"recurring documents {mask} D={D}")
    finally:
        fb.fl_set_tuning("bwd_wg_target", 0)
