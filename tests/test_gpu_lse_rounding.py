"""The last bit of the forward kernels' lse: reference times ln 2, rounded, plus the logarithm of the row sum, rounded.  The gradients follow
it (P is formed from lse), so it is the same in kernels of every shape."""
import numpy as np
import pytest

from paper_2511_02043_amd import inputs, runner

pytestmark = pytest.mark.gpu

LN2 = np.float32(np.log(2.0))


# four and eight waves, one and two row blocks, pairs of q-tiles, other head dims
@pytest.mark.parametrize("B,H,S,D,causal", [(1, 2, 70, 32, False), (1, 2, 70, 64, False), (4, 16, 700, 64, False), (2, 4, 70, 128, False), (4, 32, 1025, 128, True)])
def test_two_equal_scores(B, H, S, D, causal):
    """Two keys with the same power of two as their score: the reference is that power times log2(e), exactly its fp32 value, the sum 2."""
    import torch
    w = inputs.causal_bf16(B=B, H=H, S=S, Sk=2, D=D, causal=causal)
    w.scale = 0.1234
    w.q_offset = 2
    power = np.arange(S) % 12 - 4
    w.q[...] = 0
    w.q[..., 0] = np.exp2(power).astype(np.float32) * np.where(np.arange(S) % 5 == 0, -1, 1)
    w.k[...] = 0
    w.k[..., 0] = 1
    dw = runner.upload(w)
    dw.run_checked()
    torch.cuda.synchronize()
    reference = w.q[..., 0] * (np.float32(w.scale) * np.float32(1.4426950408889634))
    expect = reference * LN2 + LN2                 # numpy rounds the product and the sum
    fused = (reference.astype(np.float64) * np.float64(LN2) + np.float64(LN2)).astype(np.float32)
    assert np.any(expect != fused)
    assert np.array_equal(dw.lse.cpu().numpy().reshape(expect.shape), expect.astype(np.float32))
