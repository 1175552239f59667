"""The work that a user of this library has it do, as a fixed list of timed cases.

Every case goes through the public entry points: `attention()`, `variant_attention()`, `decode_attention()` and
`paged_prefill_attention()` of `paper_2511_02043_amd.functional`, and the C ABI through `paper_2511_02043_amd.binding`
where that is the only way to a path (fp32 storage, variants compiled from expressions).  Shapes are the benchmark
configurations of this repository (`paper_2511_02043_amd/inputs.py`), its paper grid, or generic ones.

`listed()` is the list, `draw(rng)` one more case of the ranges that it stands for, `prepare(case, seed)` what a program
holds before the call, `run(state)` one pass, `work(case)` the bytes and operations a pass cannot do without,
`tolerance(case)` how far another correct implementation may be.
"""
import functools

import numpy as np
import torch

from paper_2511_02043_amd import binding as fb
from paper_2511_02043_amd import functional as fn

DEVICE = "cuda:0"
_MOST_FLOPS = 3.9e12                  # no drawn case costs more than the largest listed one
_MOST_BYTES = 2.2e9                   # ... nor moves more than the listed decode step


def listed():
    return [
        # a short prompt of a small model: one launch of a few workgroups, bound by latency and the host path
        dict(name="fwd_small", kind="attention", grad=False, variant="causal", B=1, H=8, Hkv=8, S=128, D=64),
        # the headline configuration: causal self-attention over long sequences
        dict(name="fwd_causal_d128", kind="attention", grad=False, variant="causal", B=4, H=16, Hkv=16, S=8192, D=128),
        # soft-capped scores, no mask, a sequence length that no tile divides
        dict(name="fwd_softcap_d64_ragged", kind="attention", grad=False, variant="softcap", B=8, H=16, Hkv=16, S=1999, D=64),
        # a training step of a grouped-query decoder layer (the largest case)
        dict(name="train_causal_gqa_d128", kind="attention", grad=True, variant="causal", B=2, H=32, Hkv=8, S=8192, D=128),
        # training on packed documents with a sliding window (per-token document ids)
        dict(name="train_window_doc_d64", kind="attention", grad=True, variant="window_doc", B=8, H=16, Hkv=16, S=2048, D=64),
        # training of differential attention with the sub-layer RMSNorm: two softmax streams over one set of values
        dict(name="train_diff_rms", kind="differential", grad=True, B=2, H=16, S=4096, D=64, Dv=128),
        # training of Evoformer row-wise gated attention: pair bias, per-row key bias, gate, head dim 32
        dict(name="train_evoformer", kind="evoformer", grad=True, B=1, Nseq=128, Nres=384, H=8, D=32, biases=1),
        # one decode step of a full serving batch over a paged cache
        dict(name="decode_batch", kind="decode", B=64, H=32, Hkv=8, D=128, lo=4096, hi=8192, page=16),
        # one decode step of a single short conversation: latency
        dict(name="decode_single", kind="decode", B=1, H=32, Hkv=8, D=64, lo=1500, hi=2000, page=16),
        # a chunk of prompt tokens per sequence against the same kind of cache (chunked prefill)
        dict(name="prefill_chunk", kind="prefill", B=8, H=32, Hkv=8, D=128, Sq=512, lo=4096, hi=8192, page=16),
        # fp32 storage, where a user wants fp32 results
        dict(name="fwd_f32", kind="f32", causal=False, B=2, H=8, S=1024, D=64),
        # a variant given as expressions that read captured tensors: document mask and a learned relative-position bias
        dict(name="fwd_expression", kind="expression", B=4, H=16, S=4096, D=64, docs=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= _MOST_FLOPS and w["bytes"] <= _MOST_BYTES:
            return case


def _draw(rng):
    kind = rng.choice(["attention", "attention", "attention_grad", "attention_grad", "differential", "evoformer", "decode",
                       "decode", "prefill", "f32", "expression"])
    if kind in ("attention", "attention_grad"):
        D = rng.choice([64, 128])
        H, Hkv = rng.choice([(8, 8), (16, 16), (16, 2), (32, 8)])
        S = _log_int(rng, 64, 16384)
        B = max(1, min(64, _log_int(rng, 1, max(1, 32768 // S))))
        variant = rng.choice(["plain", "causal", "alibi", "softcap", "window", "prefix", "document", "window_doc"])
        return dict(kind="attention", grad=kind == "attention_grad", variant=variant, B=B, H=H, Hkv=Hkv, S=S, D=D)
    if kind == "differential":
        S = _log_int(rng, 128, 4096)
        return dict(kind="differential", grad=rng.choice([False, True]), B=rng.choice([1, 2, 4]), H=rng.choice([8, 16]), S=S,
                    D=64, Dv=128)
    if kind == "evoformer":
        return dict(kind="evoformer", grad=rng.choice([False, True]), B=1, Nseq=_log_int(rng, 16, 256),
                    Nres=_log_int(rng, 64, 512), H=rng.choice([4, 8]), D=rng.choice([32, 64]), biases=rng.choice([1, 2]))
    if kind == "decode":
        hi = _log_int(rng, 128, 32768)
        return dict(kind="decode", B=_log_int(rng, 1, 128), H=32, Hkv=8, D=rng.choice([64, 128]), lo=max(1, hi // 2), hi=hi, page=16)
    if kind == "prefill":
        Sq = _log_int(rng, 32, 2048)
        hi = _log_int(rng, 2 * Sq, 16384)
        return dict(kind="prefill", B=_log_int(rng, 1, 16), H=32, Hkv=8, D=128, Sq=Sq, lo=max(Sq, hi // 2), hi=hi, page=16)
    if kind == "f32":
        return dict(kind="f32", causal=rng.choice([False, True]), B=rng.choice([1, 2]), H=rng.choice([2, 8]),
                    S=_log_int(rng, 64, 2048), D=rng.choice([32, 64, 128]))
    return dict(kind="expression", B=rng.choice([1, 2, 4]), H=16, S=_log_int(rng, 512, 4096), D=rng.choice([64, 128]), docs=12)


# ---- inputs -----------------------------------------------------------------------------------------------------------

_WINDOW, _PREFIX, _CAP, _REL = 512, 256, 30.0, 128


def _normal(gen, *shape, dtype=torch.bfloat16):
    """N(0, 1), drawn in fp32 and rounded to the storage type."""
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32).to(dtype)


def _run_lengths(batch, seq, seed, lo=64, hi=1024):
    """Document ids of packed sequences: run lengths uniform on [lo, hi], the last run cut."""
    rng = np.random.default_rng(seed)
    ids = np.empty((batch, seq), np.int32)
    for b in range(batch):
        cuts = np.cumsum(rng.integers(lo, hi + 1, size=seq // lo + 1))
        ids[b] = np.searchsorted(cuts, np.arange(seq), side="right")
    return ids


def _fixed_count(batch, seq, docs, seed):
    """Document ids with a fixed number of documents per sequence, cut points uniform."""
    rng = np.random.default_rng(seed)
    ids = np.empty((batch, seq), np.int32)
    for b in range(batch):
        cuts = np.sort(rng.choice(np.arange(1, seq), size=min(docs, seq) - 1, replace=False))
        ids[b] = np.searchsorted(cuts, np.arange(seq), side="right")
    return ids


def _doc_ids(case, seed):
    if case.get("variant") == "window_doc":
        return _run_lengths(case["B"], case["S"], seed)
    return _fixed_count(case["B"], case["S"], case.get("docs", 12), seed)


def _slopes(H):
    return torch.tensor([2.0 ** (-8.0 * (h + 1) / H) for h in range(H)], dtype=torch.float32, device=DEVICE)


def _prepare_attention(case, seed, gen):
    B, H, Hkv, S, D = (case[n] for n in ("B", "H", "Hkv", "S", "D"))
    q, k, v = _normal(gen, B, H, S, D), _normal(gen, B, Hkv, S, D), _normal(gen, B, Hkv, S, D)
    options = {}
    variant = case["variant"]
    if variant == "causal":
        options["causal"] = True
    elif variant == "alibi":
        options["alibi_slopes"] = _slopes(H)
    elif variant == "softcap":
        options["softcap"] = _CAP
    elif variant in ("window", "window_doc"):
        options["window"] = _WINDOW
    elif variant == "prefix":
        options["prefix"] = min(_PREFIX, S)
    if variant in ("document", "window_doc"):
        options["q_doc_ids"] = torch.from_numpy(_doc_ids(case, seed)).to(DEVICE)
    state = dict(inputs=[q, k, v], options=options)
    if case["grad"]:
        state["dout"] = _normal(gen, B, H, S, D)
    return state


def _prepare_differential(case, seed, gen):
    B, H, S, D, Dv = (case[n] for n in ("B", "H", "S", "D", "Dv"))
    q_all, k_all = _normal(gen, B, 2 * H, S, D), _normal(gen, B, 2 * H, S, D)      # one projection, two streams
    q, q2 = q_all[:, :H], q_all[:, H:]
    k, k2 = k_all[:, :H], k_all[:, H:]
    v = _normal(gen, B, H, S, Dv)
    lam = torch.full((H,), 0.8, device=DEVICE)
    weight = 1.0 + 0.1 * torch.randn(Dv, generator=gen, device=DEVICE)
    state = dict(inputs=[q, k, v, q2, k2, lam, weight], names=["q2", "k2", "lam", "rms_weight"],
                 options=dict(causal=True, rmsnorm=True))
    if case["grad"]:
        state["dout"] = _normal(gen, B, H, S, Dv)
    return state


def _prepare_evoformer(case, seed, gen):
    B, Nseq, Nres, H, D = (case[n] for n in ("B", "Nseq", "Nres", "H", "D"))
    act = lambda: _normal(gen, B, Nseq, Nres, H, D).transpose(2, 3)                # storage [B, Nseq, Nres, H, D]
    q, k, v, gate = act(), act(), act(), act()
    biases = [_normal(gen, B, 1, H, Nres, Nres)]
    if case["biases"] == 2:
        biases.append(_normal(gen, B, Nseq, 1, 1, Nres))
    state = dict(inputs=[q, k, v, gate] + biases, names=["gate"], biases=len(biases), options={})
    if case["grad"]:
        state["dout"] = act()
    return state


def _prepare_cache(case, seed, gen):
    """A paged cache whose pages are handed out in arbitrary order, as a serving system's allocator does."""
    B, H, Hkv, D, page = (case[n] for n in ("B", "H", "Hkv", "D", "page"))
    rng = np.random.default_rng(seed)
    lens = rng.integers(case["lo"], case["hi"] + 1, size=B).astype(np.int32)
    per_seq = -(-case["hi"] // page)
    table = rng.permutation(B * per_seq).astype(np.int32).reshape(B, per_seq)
    k_cache, v_cache = (_normal(gen, B * per_seq, page, Hkv, D) for _ in range(2))
    q = _normal(gen, B, H, D) if case["kind"] == "decode" else _normal(gen, B, H, case["Sq"], D)
    return dict(q=q, k_cache=k_cache, v_cache=v_cache, lens=torch.from_numpy(lens).to(DEVICE),
                table=torch.from_numpy(table).to(DEVICE), max_len=case["hi"])


def _prepare_f32(case, seed, gen):
    B, H, S, D = (case[n] for n in ("B", "H", "S", "D"))
    q, k, v = (_normal(gen, B, 1, H, S, D, dtype=torch.float32) for _ in range(3))
    return dict(q=q, k=k, v=v, desc=fb.variant_desc(scale=D ** -0.5, mask=fb.FL_MASK_CAUSAL if case["causal"] else 0))


@functools.lru_cache(maxsize=None)
def _expression(D):
    """Compiled once per head dim and kept, as a program keeps it: a document mask over captured ids under a causal base
    mask, and a learned bias by head and clipped distance."""
    status, handle = fb.fl_compile_variant_aux(f"s + aux2[h * {_REL} + (i - j < {_REL} ? (i - j > 0 ? i - j : 0) : {_REL - 1})]",
                                               "aux0[b * Sq + i] != aux1[b * Sk + j]", D,
                                               (fb.FL_I32, fb.FL_I32, fb.FL_BF16), fb.FL_MASK_CAUSAL)
    fb.check(status)
    return handle


def _prepare_expression(case, seed, gen):
    B, H, S, D = (case[n] for n in ("B", "H", "S", "D"))
    q, k, v = (_normal(gen, B, 1, H, S, D) for _ in range(3))
    ids = torch.from_numpy(_doc_ids(case, seed)).to(DEVICE)
    bias = 0.5 * torch.randn(H, _REL, generator=gen, device=DEVICE)
    return dict(q=q, k=k, v=v, handle=_expression(D), aux=(ids, ids, bias.to(torch.bfloat16)), scale=D ** -0.5)


_PREPARE = dict(attention=_prepare_attention, differential=_prepare_differential, evoformer=_prepare_evoformer,
                decode=_prepare_cache, prefill=_prepare_cache, f32=_prepare_f32, expression=_prepare_expression)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    state = _PREPARE[case["kind"]](case, seed, gen)
    state["kind"] = case["kind"]
    if "inputs" in state and "dout" in state:
        for x in state["inputs"]:
            x.requires_grad_(True)
    return state


# ---- one pass ---------------------------------------------------------------------------------------------------------

def _step(state, out):
    """A training step's part: the output and the gradient of every input."""
    if "dout" not in state:
        return out
    return (out,) + torch.autograd.grad(out, state["inputs"], state["dout"])


def _run_functional(state):
    x, options = state["inputs"], state["options"]
    if state["kind"] == "attention":
        return _step(state, fn.attention(*x, **options))
    named = dict(zip(state.get("names", ()), x[3:]))
    biases = x[len(x) - state.get("biases", 0):]
    return _step(state, fn.variant_attention(*x[:3], **named, biases=biases, **options))


def _run_decode(state):
    return fn.decode_attention(state["q"], state["k_cache"], state["v_cache"], state["lens"], state["table"],
                               max_seq_len=state["max_len"])


def _run_prefill(state):
    return fn.paged_prefill_attention(state["q"], state["k_cache"], state["v_cache"], state["lens"], state["table"],
                                      max_seq_len=state["max_len"])


def _run_f32(state):
    q = state["q"]
    out = torch.empty_like(q)
    lse = torch.empty(q.shape[:-1] + (1,), dtype=torch.float32, device=q.device)
    fb.check(fb.fl_attn_fwd(*(fb.tensor_desc(state[n]) for n in "qkv"), state["desc"], None, fb.tensor_desc(out),
                            fb.tensor_desc(lse), torch.cuda.current_stream().cuda_stream))
    return out, lse


def _run_expression(state):
    q = state["q"]
    out = torch.empty_like(q)
    lse = torch.empty(q.shape[:-1] + (1,), dtype=torch.float32, device=q.device)
    tq, tk, tv = (fb.tensor_desc(state[n]) for n in "qkv")
    ws = torch.empty(fb.fl_custom_skip_workspace_size(state["handle"], tq, tk), dtype=torch.uint8, device=q.device)
    fb.check(fb.fl_attn_fwd_custom_skip(state["handle"], tq, tk, tv, state["scale"], state["aux"], ws, fb.tensor_desc(out),
                                        fb.tensor_desc(lse), torch.cuda.current_stream().cuda_stream))
    return out, lse


_RUN = dict(attention=_run_functional, differential=_run_functional, evoformer=_run_functional, decode=_run_decode,
            prefill=_run_prefill, f32=_run_f32, expression=_run_expression)


def run(state):
    return _RUN[state["kind"]](state)


# ---- work and tolerance -----------------------------------------------------------------------------------------------

def _causal_pairs(S, window=None):
    if window is None or window >= S:
        return S * (S + 1) / 2
    return (window + 1) * S - window * (window + 1) / 2


def _document_pairs(ids, window, causal):
    """Visible (i, j) pairs of one head, summed over the batch: j in i's document and, where asked for, at most `window`
    before i."""
    total = 0.0
    for row in ids:
        for n in np.unique(row, return_counts=True)[1]:
            total += _causal_pairs(int(n), window) if causal else float(n) ** 2
    return total


def _pairs(case):
    """Visible (query, key) pairs of one head, summed over the batch (document masks: those of one seed)."""
    B, S, variant = case["B"], case["S"], case.get("variant", "causal")
    if case["kind"] == "expression":
        return _document_pairs(_doc_ids(case, 0), None, True)
    if variant == "window_doc":
        return _document_pairs(_doc_ids(case, 0), _WINDOW, True)
    if variant == "document":
        return _document_pairs(_doc_ids(case, 0), None, False)
    if variant == "causal":
        return B * _causal_pairs(S)
    if variant == "window":
        return B * _causal_pairs(S, _WINDOW)
    if variant == "prefix":
        return B * (_causal_pairs(S) + min(_PREFIX, S) * (min(_PREFIX, S) - 1) / 2)
    return B * float(S) ** 2


def work(case):
    """Each input read once and each output written once; two contractions per visible score in the forward pass and five
    in the backward pass (the scores again, dP, dV, dQ, dK)."""
    kind = case["kind"]
    if kind == "attention":
        B, H, Hkv, S, D = (case[n] for n in ("B", "H", "Hkv", "S", "D"))
        pairs = _pairs(case) * H
        q_bytes, kv_bytes = 2 * B * H * S * D, 2 * B * Hkv * S * D
        if case["grad"]:                           # in: q, k, v, dout; out: out, dq, dk, dv
            return dict(bytes=4 * q_bytes + 4 * kv_bytes, flops=14 * D * pairs)
        return dict(bytes=2 * q_bytes + 2 * kv_bytes, flops=4 * D * pairs)
    if kind == "differential":
        B, H, S, D, Dv = (case[n] for n in ("B", "H", "S", "D", "Dv"))
        pairs = 2 * B * H * _causal_pairs(S)
        qk, vo = 4 * 2 * B * H * S * D, 2 * B * H * S * Dv                         # q, k, q2, k2; one tensor of v's size
        if case["grad"]:
            return dict(bytes=2 * qk + 4 * vo, flops=(8 * D + 6 * Dv) * pairs)
        return dict(bytes=qk + 2 * vo, flops=(2 * D + 2 * Dv) * pairs)
    if kind == "evoformer":
        B, Nseq, Nres, H, D = (case[n] for n in ("B", "Nseq", "Nres", "H", "D"))
        act, pair = 2 * B * Nseq * Nres * H * D, 2 * B * H * Nres * Nres
        key = 2 * B * Nseq * Nres if case["biases"] == 2 else 0
        scores = B * Nseq * H * float(Nres) ** 2
        if case["grad"]:                           # in: q, k, v, gate, dout; out: out and four gradients
            return dict(bytes=10 * act + 2 * (pair + key), flops=14 * D * scores)
        return dict(bytes=5 * act + pair + key, flops=4 * D * scores)
    if kind in ("decode", "prefill"):
        B, H, Hkv, D = (case[n] for n in ("B", "H", "Hkv", "D"))
        tokens = B * (case["lo"] + case["hi"]) / 2
        Sq = case.get("Sq", 1)
        return dict(bytes=2 * 2 * tokens * Hkv * D + 2 * 2 * B * H * Sq * D,
                    flops=4 * D * H * B * Sq * ((case["lo"] + case["hi"]) / 2 - (Sq - 1) / 2))
    B, H, S, D = (case[n] for n in ("B", "H", "S", "D"))
    if kind == "f32":
        pairs = B * H * (_causal_pairs(S) if case["causal"] else float(S) ** 2)
        return dict(bytes=4 * 4 * B * H * S * D, flops=4 * D * pairs)
    return dict(bytes=4 * 2 * B * H * S * D, flops=4 * D * H * _pairs(case))


def tolerance(case):
    """Against an fp64 evaluation the bf16 paths measure 1.7e-3 (a differential forward pass) to 3.5e-3 (the gradients of the
    biases and of the differential values), the rounding of the outputs and of P and dS to bf16; fp32 storage 2.8e-7."""
    if case["kind"] == "f32":
        return dict(rel=2e-6)
    return dict(rel=1e-2)
