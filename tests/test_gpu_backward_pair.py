"""The stationary-bias backward kernels (a pair bias shared by the row problems, with or without a key bias): dQ, dK, dV and both
bias gradients against the fp64 oracle where tiles end -- 32-row blocks, 64 owned rows, steps of 128 streamed rows, ranges of the
row axis -- and against the general kernels; the tuning switch selects either for calls of any size.  Tolerance: fl_attn_bwd_ex's
(P and dS in bf16, fp32 sums; relative L2 <= 5e-3)."""
import numpy as np
import pytest
import torch

from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import inputs, runner
from test_gpu_backward_ex import compare

pytestmark = pytest.mark.gpu

C = inputs.combination_bf16
PAIR, GENERAL = 2, 1                               # the tuning switch: always these kernels, never


@pytest.fixture
def always_pair():
    fb.check(fb.fl_set_tuning("pair_bias", PAIR))
    yield
    fb.fl_set_tuning("pair_bias", 0)


@pytest.mark.parametrize("n_bias", [1, 2])
@pytest.mark.parametrize("D,Sq,Sk,G,H", [(32, 1, 1, 2, 1), (32, 31, 33, 3, 2), (32, 64, 128, 9, 1), (32, 65, 129, 2, 2), (32, 257, 200, 3, 1), (32, 384, 300, 2, 2),
                                         (32, 385, 511, 2, 1), (32, 512, 40, 2, 1), (64, 33, 64, 5, 2), (64, 128, 65, 2, 2), (64, 129, 256, 3, 1), (64, 256, 257, 2, 1), (64, 300, 384, 2, 1)])
def test_sizes(D, Sq, Sk, G, H, n_bias, always_pair):
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
    new, old = _grads(w, dout, PAIR, dtype), _grads(w, dout, GENERAL, dtype)
    assert new.keys() == old.keys() and any(n.startswith("dbias") for n in new)
    for n in new:
        assert np.all(np.isfinite(new[n])), n
        rel = np.linalg.norm(new[n] - old[n]) / np.linalg.norm(old[n])
        print(f"{form} D {D} {n}: {rel:.2e}", flush=True)
        assert rel <= 4e-3, n                      # both round P and dS to bf16 (2^-9 each)
    assert not all(np.array_equal(new[n], old[n]) for n in new), "the switch chose the same kernels"


# half of the compute units or a narrow tensor: the general kernels (two row problems, up to 64 rows, one query row, a last round of
# workgroups that is nearly empty); enough row problems, and launches that are small for either
@pytest.mark.parametrize("B,G,H,Sq,Sk,route", [(8, 2, 8, 200, 200, GENERAL), (1, 64, 4, 64, 64, GENERAL), (4, 16, 4, 1, 200, GENERAL), (4, 16, 4, 200, 1, GENERAL),
                                               (10, 6, 8, 96, 96, GENERAL), (1, 128, 8, 96, 80, PAIR), (1, 128, 4, 200, 130, PAIR), (1, 6, 4, 100, 72, PAIR)])
def test_route(B, G, H, Sq, Sk, route):
    """Which kernels a call takes without the tuning switch: the general ones give the same bits with and without it."""
    w = C(D=32, n_bias=1, S=Sq, Sk=Sk, G=G, B=B, H=H)
    w.biases = (w.biases[0][:, :1],)
    dout = inputs.dout_for(w)
    got, general = _grads(w, dout, 0), _grads(w, dout, GENERAL)
    assert all(np.array_equal(got[n], general[n]) for n in got) == (route == GENERAL)


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
    g = _grads(w, inputs.dout_for(w), PAIR)
    for n, x in g.items():
        assert np.all(np.isfinite(x)), n
    assert np.all(g["dk0"][0, 0, :, 100:] == 0) and np.all(g["dv0"][0, 0, :, 100:] == 0) and np.all(g["dk0"][0, 2, :, :70] == 0)
    assert np.any(g["dk0"][0, 0, :, :100] != 0) and np.any(g["dk0"][0, 2, :, 70:] != 0)
    if np.isinf(hide):
        assert all(np.all(g[n][0, 4] == 0) for n in ("dq0", "dk0", "dv0"))
    old = _grads(w, inputs.dout_for(w), GENERAL)
    for n in g:
        assert np.linalg.norm(g[n] - old[n]) <= 4e-3 * np.linalg.norm(old[n]), n


def _workload_with_hidden(D, value, by):
    """Six row problems; all keys of row problem 4 (by a key bias) or of query row 7 (by the pair bias) get `value`, the rest of both
    biases as drawn."""
    w = inputs.evoformer_bf16(B=1, Nseq=6, Nres=150, H=2, D=D, two_biases=True, salt=9)
    pair, key = (x.copy() for x in w.biases)
    if by == "key":
        key[0, 4] = value
    else:
        pair[0, 0, :, 7] = value
    w.biases = (inputs.round_to_bf16(pair), inputs.round_to_bf16(key))
    dout = inputs.dout_for(w)
    rows = (0, 4) if by == "key" else (0, slice(None), slice(None), 7)     # of q, dq and dout
    return w, dout, rows


# bf16 numbers at which lse * log2(e) and bias * log2(e) differ by up to a unit in the last place of numbers of that size (128 near
# 1e9, far beyond what exp2 takes), larger ones, and half of the type's lowest value
LARGE = [-1e4, -1e9, -7.93e8, -3.1e9, -1e10, -1e20, -1e38, -1.69e38]


@pytest.mark.parametrize("tune", [PAIR, GENERAL])
@pytest.mark.parametrize("by", ["key", "pair"])
@pytest.mark.parametrize("value", LARGE)
@pytest.mark.parametrize("D", [32, 64])
def test_rows_hidden_by_finite_bias(D, value, by, tune):
    """A row all of whose keys are hidden by a large finite bias (padding).  Its lse is that bias up to rounding; P is at most 1 all
    the same.  Where its dO is zero it contributes nothing to any gradient; else the contribution is finite and bounded."""
    w, dout, rows = _workload_with_hidden(D, value, by)
    full = _grads(w, dout, tune)
    silent = dout.copy()
    silent[rows] = 0
    got = _grads(w, silent, tune)
    dead, _, _ = _workload_with_hidden(D, -np.inf, by)
    want = _grads(dead, silent, tune)               # P = 0 there: the sums over the other rows alone
    for n in got:
        assert np.all(np.isfinite(full[n])) and np.all(np.isfinite(got[n])), n
        assert np.array_equal(got[n], want[n]), n
    assert np.all(got["dq0"][rows] == 0)
    if by == "key":                                # |dV| <= sum over the queries of P |dO| with P <= 1, dO and P rounded to bf16
        bound = np.abs(dout[0, 4]).sum(axis=1, keepdims=True)
        assert np.all(np.abs(full["dv0"][0, 4]) <= bound * (1 + 2.0 ** -6))


@pytest.mark.parametrize("offset", [0.0, -30.0, -1e4])
@pytest.mark.parametrize("D,n_bias", [(32, 1), (32, 2), (64, 1), (64, 2)])
def test_exponents_are_those_of_the_general_kernels(D, n_bias, offset):
    """The exponent of every score is formed as in the general kernels, so an offset that all keys of a row share costs no more
    than it does there.  What may differ: delta enters in front of the sum over the channels instead of behind it, 2^-24 of
    |delta| + |dP|, which turns the bf16 rounding (2^-8 apart) of about one dS in 2^14 by 2^-8: 2^-15 of the norm; bound 1e-4."""
    w = inputs.evoformer_bf16(B=1, Nseq=5, Nres=150, H=2, D=D, two_biases=n_bias == 2, salt=4)
    if offset:                                     # (-1e4 and normal numbers have no sum in bf16: the last bias is the offset alone)
        w.biases = w.biases[:-1] + (inputs.round_to_bf16(np.full_like(w.biases[-1], offset)),)
    dout = inputs.dout_for(w)
    new, old = _grads(w, dout, PAIR), _grads(w, dout, GENERAL)
    for n in ("dq0", "dk0", "dv0", "dbias0"):
        rel = np.linalg.norm(new[n] - old[n]) / np.linalg.norm(old[n])
        print(f"D {D} biases {n_bias} offset {offset} {n}: {rel:.2e}", flush=True)
        assert rel <= 1e-4, n


def test_nan_stays_where_it_is():
    """A NaN bias value and a NaN in V spoil the same gradients as with the general kernels, no more and no fewer."""
    w = inputs.evoformer_bf16(B=1, Nseq=4, Nres=70, H=2, D=32, salt=3)
    pair, v = w.biases[0].copy(), w.v.copy()
    pair[0, 0, 0, 5, 9] = np.nan
    v[0, 2, 1, 40, 3] = np.nan
    w.biases, w.v = (pair,), v
    dout = inputs.dout_for(w)
    new, old = _grads(w, dout, PAIR), _grads(w, dout, GENERAL)
    for n in new:
        assert np.array_equal(np.isnan(new[n]), np.isnan(old[n])), n
    assert np.isnan(new["dq0"][0, 0, 0, 5]).all() and not np.isnan(new["dq0"][0, 0, 0, 6]).any()


def _call(x, biases, dbias, D):
    """Gradients of q, k, v (dense) and of the biases (into `dbias`) from x = q, k, v, dout and biases in any layout.  The forward
    pass, which wants biases with unit key stride, runs on dense copies."""
    q, k, v, dout = x
    desc = fb.variant_desc(scale=D ** -0.5, n_bias=len(biases))
    out = torch.empty(q.shape, dtype=torch.bfloat16, device=q.device)
    lse = torch.empty(q.shape[:-1] + (1,), device=q.device)
    t = fb.tensor_desc
    ws = torch.empty(fb.fl_attn_bwd_ex_workspace_size(t(q), t(k), t(v), desc), dtype=torch.uint8, device=q.device)
    dense = [y.contiguous() for y in (q, k, v, *biases)]
    fb.check(fb.fl_attn_fwd(*(t(y) for y in dense[:3]), desc, fb.aux_desc(biases=dense[3:]), t(out), t(lse), 0))
    g = [torch.full(y.shape, float("nan"), device=q.device) for y in (q, k, v)]
    fb.check(fb.fl_attn_bwd_ex(t(q), t(k), t(v), t(out), t(dout), t(lse), desc, fb.aux_desc(biases=biases, workspace=ws), *(t(y) for y in g),
                               fb.bwd_extra(dbias=dbias), 0))
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("form", ["bias_by_columns", "bias_rows_apart", "strided_bias_gradients", "far_rows"])
@pytest.mark.parametrize("D", [32, 64])
def test_layouts(D, form, always_pair):
    """The same numbers in other layouts give the same bits: a pair bias whose query axis is the contiguous one (no wide loads in either
    kernel) or whose rows are an odd number of elements apart, bias gradients stored with gaps and transposed, rows of
    q, k, v and dout 8 MB apart."""
    B, G, H, Sq, Sk = 2, 5, 2, 70, 150
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda:0").to(torch.bfloat16)
    x = [rand(B, G, H, s, D) for s in (Sq, Sk, Sk, Sq)]
    biases = [rand(B, 1, H, Sq, Sk), rand(B, G, 1, 1, Sk)]
    dbias = [torch.full(b.shape, float("nan"), device=b.device) for b in biases]
    want = _call(x, biases, dbias, D)
    pair, key = biases
    if form == "bias_by_columns":
        biases = [pair.transpose(3, 4).contiguous().transpose(3, 4), key]
    elif form == "bias_rows_apart":
        wide = rand(B, 1, H, Sq, Sk + 7)
        wide[..., 3:Sk + 3] = pair
        biases = [wide[..., 3:Sk + 3], rand(B, G, 1, 1, 3 * Sk)[..., ::3].copy_(key)]
    elif form == "far_rows":
        far = []
        for y in x:
            store = torch.empty(y.shape[3], 1 << 22, dtype=torch.bfloat16, device="cuda:0")
            view = store[:, :B * G * H * D].view(y.shape[3], B, G, H, D).permute(1, 2, 3, 0, 4)
            far.append(view.copy_(y))
        x = far
    got_db = [torch.full(b.shape, float("nan"), device=b.device) for b in biases]
    if form == "strided_bias_gradients":
        got_db = [torch.full((B, 1, H, Sk, 2 * Sq), float("nan"), device="cuda:0")[..., ::2].transpose(3, 4),
                  torch.full((B, G, 1, 1, 5 * Sk), float("nan"), device="cuda:0")[..., 1::5]]
    got = _call(x, biases, got_db, D)
    for a, b in zip(want + dbias, got + got_db):
        assert torch.isfinite(b).all() and torch.equal(a, b)
