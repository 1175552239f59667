"""Decode workgroups of fewer waves, which launches of more than 256 workgroups with short key ranges take: lengths around tiles and
around the rounds of one, two and four waves, empty sequences, score_mods and windows; against the fp64 oracle (tolerance of
test_gpu_decode.py)."""
import numpy as np
import pytest

from paper_2511_02043_amd import inputs
from tests.test_gpu_decode import compare

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 63, 65, 96, 127, 128, 129, 160, 161, 255, 257]


def lengths(B, longest):
    rng = np.random.default_rng(B)
    lens = rng.integers(0, longest + 1, size=B)
    edges = [n for n in EDGES if n <= longest] + [longest]
    lens[:len(edges)] = edges
    return lens


# sequences, kv heads, head dim, longest sequence: two and four waves at head dim 64, one, two and five at 128
@pytest.mark.parametrize("B,Hkv,D,longest", [
    (65, 8, 64, 300), (65, 8, 64, 512), (33, 8, 64, 300), (129, 4, 128, 300), (129, 4, 128, 513), (33, 8, 128, 300), (33, 8, 128, 545),
])
def test_decode_waves(B, Hkv, D, longest):
    compare(inputs.decode_bf16(H=2 * Hkv, Hkv=Hkv, D=D, page_size=16, seq_lens=lengths(B, longest), salt=7), f"{B}x{Hkv}x{longest}")


@pytest.mark.parametrize("B,D", [(65, 64), (33, 64), (65, 128), (33, 128)])
@pytest.mark.parametrize("variant", ["softcap", "alibi_window", "bf16"])
def test_decode_waves_variants(B, D, variant):
    w = inputs.decode_bf16(H=16, Hkv=8, D=D, page_size=32, seq_lens=lengths(B, 200), salt=8)
    if variant == "softcap":
        w.softcap = 2.0
    elif variant == "alibi_window":
        w.alibi = inputs.alibi_slopes(16)
        w.window = 70
    compare(w, variant, out_dtype="bf16" if variant == "bf16" else "f32")


@pytest.mark.parametrize("B,D,window", [(33, 64, 40), (65, 64, 255), (33, 128, 40), (65, 128, 255), (33, 128, 600)])
def test_decode_waves_window(B, D, window):
    """Long sequences of which a workgroup sees a window's tiles only: fewer waves, as for short ones."""
    lens = np.random.default_rng(B).integers(1, 1301, size=B)
    lens[:8] = [0, 1, 31, window, window + 1, window + 33, 1299, 1300]
    w = inputs.decode_bf16(H=16, Hkv=8, D=D, page_size=16, seq_lens=lens, salt=9)
    w.window = window
    compare(w, f"window {window}")
