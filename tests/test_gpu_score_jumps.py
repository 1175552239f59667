"""Scores that rise along the keys: the forward kernels without ALiBi, biases or window take a tile's exponentials against what the row's
reference was before it, let the reference follow the row sums, and run a q-tile again with the max of every tile where something
overflowed on the way.  Against the fp64 oracle."""
import numpy as np
import pytest

from oracle import attention_oracle as ao
from oracle import decode_oracle as do
from paper_2511_02043_amd import inputs, runner
from tests.gpu_util import TOL, errors, lse_error

pytestmark = pytest.mark.gpu


# level (natural log) by key, as a function of j / Sk
LEVELS = {
    "ramp": lambda x, n: 70.0 * x,                                   # the reference follows, tile by tile
    "step": lambda x, n: np.where(x < 0.5, 0.0, 60.0),               # ... once, by 2^86
    "far": lambda x, n: np.where(x < 0.5, 0.0, 76.0),                # ... by 2^110
    "jump": lambda x, n: np.where(x < 0.5, 0.0, 120.0),              # past 2^117: the q-tile runs again
    "jumps": lambda x, n: 100.0 * np.floor(4 * x),
    "last": lambda x, n: np.where(np.arange(n) == n - 1, 300.0, 0.0),
    "down": lambda x, n: np.where(x < 0.4, 200.0, 0.0),
    "deep": lambda x, n: np.where(x < 0.7, -400.0, -100.0),
}


def raise_scores(q, k, scale, level):
    """First channel of q and k so that key j's scores carry level[j] (a value that bf16 holds: 8 x level / (8 x scale), rounded)."""
    q[..., 0] = np.float32(8.0)
    k[..., 0] = inputs.round_to_bf16((level / (8.0 * scale)).astype(np.float32))


def compare(w, unit=1.0, lse_slack=2.0 ** -15):
    import torch
    dw = runner.upload(w)
    dw.out.fill_(float("nan"))
    dw.run_checked()
    torch.cuda.synchronize()
    got, lse = dw.out.float().cpu().numpy().astype(np.float64), runner.lse_to_oracle_layout(dw)
    ref, ref_lse = ao.run_workload(w)
    assert np.all(np.isfinite(got))
    max_abs, rel = errors(got / unit, ref / unit)
    assert max_abs <= TOL["bf16"]["max_abs"] and rel <= TOL["bf16"]["rel_l2"], (max_abs, rel)
    # the scores carry the level in fp32 (half a unit in the last place of up to 300, in the product and in the sum) beside the stated tolerance
    assert lse_error(lse, ref_lse) <= TOL["bf16"]["lse"] + lse_slack


@pytest.mark.parametrize("level", sorted(LEVELS))
@pytest.mark.parametrize("part", [dict(D=64), dict(D=64, pos_mask="causal"), dict(D=128), dict(D=128, pos_mask="causal", Hkv=2), dict(D=32),
                                  dict(D=64, pos_mask="prefix"), dict(D=64, score_mod="softcap", cap=4000.0, qscale=1.0),
                                  dict(D=128, score_mod="softcap", cap=4000.0, qscale=1.0, pos_mask="causal"),
                                  dict(D=64, Dv=128, diff=True), dict(D=64, Dv=128, diff=True, rmsnorm=True)], ids=str)
def test_levels(part, level):
    w = inputs.combination_bf16(B=1, H=4, S=333, Sk=520, **part)
    rise = LEVELS[level](np.arange(520) / 520, 520)
    raise_scores(w.q, w.k, w.scale, rise)
    if w.q2 is not None:
        raise_scores(w.q2, w.k2, w.scale, rise[::-1])
    compare(w)


@pytest.mark.parametrize("B,H,Hkv,S,D", [(2, 32, 8, 1025, 128), (4, 32, 32, 700, 64), (2, 32, 4, 100, 128), (2, 16, 16, 2048, 64)])
def test_other_shapes(B, H, Hkv, S, D):
    """More workgroups: pairs of q-tiles, eight waves, two row blocks, packed heads; one (b, h) problem jumps, its neighbours do not."""
    w = inputs.causal_bf16(B=B, H=H, Hkv=Hkv, S=S, Sk=max(S, 1100), D=D)
    w.q_offset = max(S, 1100) - S
    n = w.k.shape[3]
    level = np.where(np.arange(n) < n // 2, 0.0, 130.0)
    hk = Hkv // 2
    w.q[..., 0] = np.float32(8.0)
    w.k[:, :, hk, :, 0] = inputs.round_to_bf16((level / (8.0 * w.scale)).astype(np.float32))
    compare(w)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_large_values(D, causal):
    """Sums stay below 2^100 but their products with V do not stay below 2^128."""
    w = inputs.causal_bf16(B=1, H=4, S=300, Sk=300, D=D, causal=causal)
    raise_scores(w.q, w.k, w.scale, np.where(np.arange(300) < 150, 0.0, 65.0))
    w.v = w.v * np.float32(2.0 ** 60)
    compare(w, unit=2.0 ** 60)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("part", [dict(D=64), dict(D=128), dict(D=64, score_mod="softcap", cap=4000.0, qscale=1.0), dict(D=64, Dv=128, diff=True)], ids=str)
@pytest.mark.parametrize("masked", [0, 24])
def test_one_score_beside_large_values(part, causal, masked):
    """One key 12 log2 units above its row's reference: the sum of its tile stays within the bound up to which the reference is kept, but
    2^12 times values of 2^116 is past the range.  And a key of the last tile, which is masked, from which on both seem small."""
    w = inputs.combination_bf16(B=1, H=4, S=300, Sk=300, pos_mask="causal" if causal else "none", **part)
    rise = np.log(2.0) * (np.where(np.arange(300) == 200, 12.0, 0.0) + np.where(np.arange(300) == 260, masked, 0.0))
    raise_scores(w.q, w.k, w.scale, rise)
    if w.q2 is not None:
        raise_scores(w.q2, w.k2, w.scale, rise)
    # (one key's value is most of a row's result: its weight and the result rounded to bf16, 2 x 2^-9 of at most 2, is within the 1e-2)
    w.v = np.clip(w.v, -2, 2) * np.float32(2.0 ** 116)
    compare(w, unit=2.0 ** 116)


@pytest.mark.parametrize("D", [64, 128])
def test_infinite_scores(D):
    """A score of -inf hides its key; one of +inf makes its row NaN; the other rows of the workgroup stay as they are."""
    w = inputs.causal_bf16(B=1, H=2, S=256, Sk=256, D=D, causal=False)
    w.q[:, :, :, 5, :] = 0
    w.q[:, :, :, 5, 0] = np.float32(2.0 ** 100)
    w.q[:, :, :, 9, :] = 0
    w.q[:, :, :, 9, 0] = np.float32(-2.0 ** 100)
    w.k[..., 0] = 0
    w.k[:, :, :, 200, 0] = np.float32(2.0 ** 100)
    w.q[:, :, :, [i for i in range(256) if i not in (5, 9)], 0] = 0
    import torch
    dw = runner.upload(w)
    dw.run_checked()
    torch.cuda.synchronize()
    got = dw.out.float().cpu().numpy().astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref, _ = ao.run_workload(w)
    assert np.all(np.isnan(got[:, :, :, 5]))
    rows = [i for i in range(256) if i != 5]
    assert np.all(np.isfinite(got[:, :, :, rows]))
    row9 = np.delete(w.v[0, 0, :, :, :].astype(np.float64), 200, axis=1).mean(axis=1)
    assert np.max(np.abs(got[0, 0, :, 9] - row9)) <= TOL["bf16"]["max_abs"]
    rows.remove(9)
    assert np.max(np.abs(got[:, :, :, rows] - ref[:, :, :, rows])) <= TOL["bf16"]["max_abs"]


@pytest.mark.parametrize("Sq", [96, 300])
def test_paged(Sq):
    """Keys read in place from a paged cache; one sequence jumps in its middle, one shorter than the chunk."""
    import torch
    w = inputs.prefill_paged_bf16(H=8, Hkv=2, D=128, Sq=Sq, page_size=16, seq_lens=[40, 700, 1027])
    w.q[..., 0] = np.float32(8.0)
    for b, n in enumerate(w.seq_lens):
        for j in range(n):
            level = 130.0 if b == 1 and j > 350 else 0.0
            w.k_cache[w.block_table[b, j // 16], j % 16, :, 0] = inputs.round_to_bf16(np.array([level / (8.0 * w.scale)], np.float32))[0]
    dd = runner.upload_prefill_paged(w)
    dd.run_checked()
    torch.cuda.synchronize()
    got, lse = dd.out.float().cpu().numpy()[:, 0], dd.lse.cpu().numpy()[:, 0, :, :, 0]
    ref, ref_lse = do.prefill_attention(w.q, w.k_cache, w.v_cache, w.block_table, w.seq_lens, scale=w.scale)
    dead = np.isneginf(ref_lse)
    assert np.array_equal(np.isneginf(lse), dead)
    assert np.max(np.abs(got - ref)) <= TOL["bf16"]["max_abs"]
    assert np.max(np.abs(lse[~dead] - ref_lse[~dead])) <= TOL["bf16"]["lse"]


@pytest.mark.parametrize("part", [dict(D=64), dict(D=64, pos_mask="causal"), dict(D=128), dict(D=128, pos_mask="causal"), dict(D=64, Dv=128, diff=True)], ids=str)
@pytest.mark.parametrize("deviation", [8, 25, 100])
def test_scores_far_apart(part, deviation):
    """Normal scores of a large standard deviation: rows whose max is taken tile by tile (from about 16 on), beside others.  Where two keys of a row are close at the top, a weight follows its score's error: half a unit
    in the last place of the score, in the product and in the sum."""
    w = inputs.combination_bf16(B=1, H=4, S=700, Sk=700, **part)
    # (one key may be all of a row: its weight, rounded to bf16, is within 2^-8; of a value of 1, and 1 + 0.9 times in the difference of two streams)
    w.v = np.clip(w.v, -1, 1)
    w.scale = deviation * part["D"] ** -0.5
    compare(w, lse_slack=deviation * 2.0 ** -17)
