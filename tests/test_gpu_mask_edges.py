"""Gradients, and outputs under document masks, where the first and last visible key (query row) of a lane sit on and beside the edges of the 32-row blocks and
64-row tiles, for rows and keys in the middle of the tensors and at their ends; against the fp64 backward oracle with
the bounds of test_gpu_backward.py."""
import numpy as np
import pytest

from paper_2511_02043_amd import inputs
from tests.gpu_util import run_and_compare
from tests.test_gpu_backward import compare

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 128, 400]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("pos_mask,edge", [("window", e) for e in EDGES] + [("prefix", e) for e in EDGES[1:]])
def test_mask_edges(pos_mask, edge, D):
    w = inputs.combination_bf16(D=D, pos_mask=pos_mask, window=edge, prefix=edge, B=1, H=2, S=161)
    compare(w)


@pytest.mark.parametrize("pos_mask", ["none", "causal", "window", "prefix"])
@pytest.mark.parametrize("S,Sk", [(161, 95), (95, 161), (1, 65), (65, 1)])
def test_mask_edges_with_documents(pos_mask, S, Sk):
    w = inputs.combination_bf16(D=64, pos_mask=pos_mask, doc=True, window=33, prefix=33, B=2, H=4, Hkv=2, S=S, Sk=Sk)
    compare(w)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("pos_mask", ["none", "causal", "window", "prefix"])
@pytest.mark.parametrize("lengths", [[64, 64, 33], [31, 1, 32, 97], [161], None])
def test_document_edges_forward(lengths, pos_mask, D):
    """Documents that end on and beside the edges of blocks and tiles, one document for all, and ids in no order (None)."""
    w = inputs.combination_bf16(D=D, pos_mask=pos_mask, window=40, prefix=33, B=1, H=2, S=161)
    ids = np.random.default_rng(5).integers(0, 3, 161) if lengths is None else np.repeat(np.arange(len(lengths)), lengths)
    w.q_doc = w.kv_doc = ids.astype(np.int32)[None]
    run_and_compare(w)
