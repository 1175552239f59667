"""PyTorch-facing calls of the library: `attention(q, k, v, ...)` with autograd support and
`decode_attention(...)` for one decode step over a paged cache.

Marshalling only: the forward pass is fl_attn_fwd, the backward pass fl_attn_bwd, both through
the C ABI (`_fltorch`, compiled from csrc/fl_torch.cpp, fills the descriptors); no attention arithmetic happens here and there is no fallback path.  Tensors
are [B, H, S, D] (or [B, G, H, S, D] with an extra independent row axis) bf16 CUDA tensors;
strided views are passed as they are.

`attention()`: scale, causal / sliding-window / PrefixLM / document masks, ALiBi, tanh soft-cap,
grouped-query heads, query-position offset (the variants fl_attn_bwd covers).
`variant_attention()`: the same plus additive biases, the sigmoid gate, RMSNorm and the differential
second stream, differentiable in every tensor input (fl_attn_bwd_ex).
"""
from __future__ import annotations

from typing import Optional

import torch
from torch.autograd import forward_ad

from . import binding as fb

_host_module = None


def _host():
    """The compiled marshalling module (loaded once, after the library)."""
    global _host_module
    if _host_module is None:
        fb.lib()
        try:
            from . import _fltorch
        except ImportError as e:
            raise ImportError("_fltorch.so is missing or was built for another interpreter or torch: run "
                              "make -C paper_2511_02043_amd/csrc PYTHON=<this interpreter>") from e
        _fltorch.set_check(fb.check)
        _host_module = _fltorch
    return _host_module


def _stream(t: torch.Tensor) -> int:
    return torch._C._cuda_getCurrentRawStream(t.get_device())


def _as5(x: torch.Tensor) -> torch.Tensor:
    if x.dim() == 4:
        return x.unsqueeze(1)
    if x.dim() != 5:
        raise ValueError(f"expected [B, H, S, D] or [B, G, H, S, D], got {tuple(x.shape)}")
    return x


def _check_aux(name: str, t: Optional[torch.Tensor], dtype: torch.dtype, shape, device, *, contiguous: bool = True,
               inner_unit: bool = False) -> None:
    """The C ABI reads these arrays as raw int32 / float32 memory of a fixed shape: anything else
    (torch's default int64 ids, a sliced view, a tensor on another device) would be reinterpreted
    silently, so it is refused here."""
    if t is None:
        return
    if isinstance(t, torch.Tensor) and t.dtype is dtype and t.shape == shape and t.device == device and t.is_contiguous():
        return
    if not isinstance(t, torch.Tensor):
        raise ValueError(f"{name} must be a torch.Tensor")
    if t.dtype != dtype:
        raise ValueError(f"{name} must be {dtype}, got {t.dtype}")
    if t.device != device:
        raise ValueError(f"{name} is on {t.device}, expected {device}")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} must have shape {tuple(shape)}, got {tuple(t.shape)}")
    if contiguous and not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if inner_unit and t.dim() >= 2 and t.shape[-1] > 1 and t.stride(-1) != 1:
        raise ValueError(f"{name} must have unit stride along its last axis")


def _mask_bits(causal, window, prefix, q_doc_ids):
    mask = 0
    if causal:
        mask |= fb.FL_MASK_CAUSAL
    if window is not None:
        mask |= fb.FL_MASK_WINDOW | fb.FL_MASK_CAUSAL
    if prefix is not None:
        mask |= fb.FL_MASK_PREFIX
    if q_doc_ids is not None:
        mask |= fb.FL_MASK_DOC
    return mask


def _score_mod(softcap, alibi_slopes):
    if softcap is not None and alibi_slopes is not None:
        raise ValueError("one score_mod at a time")
    return fb.FL_MOD_SOFTCAP if softcap is not None else (fb.FL_MOD_ALIBI if alibi_slopes is not None else fb.FL_MOD_NONE)


# private names of torch: where one is missing, its state counts as there and every call gets its node
_transforms_active = getattr(torch._C, "_are_functorch_transforms_active", lambda: True)
_tracing_state = getattr(torch._C, "_get_tracing_state", lambda: True)
_grad_enabled = torch.is_grad_enabled


_NO_NODE, _NATIVE_NODE, _PYTHON_NODE = range(3)


def _node_for(tensors) -> int:
    """The autograd node that a call needs.  None where it takes no part in a derivative, a transform or a trace: building one takes 3.7 us, of
    8.8 us for a call on [1, 8, 128, 64] whose kernel runs 8 us.  The compiled one for ordinary derivatives; the Python one, which
    transforms, traces and torch.compile look into, for the rest."""
    if _transforms_active() or getattr(forward_ad, "_current_level", 0) >= 0 or _tracing_state() is not None or torch.compiler.is_compiling():
        return _PYTHON_NODE
    if _grad_enabled():
        for t in tensors:
            if t is not None and t.requires_grad:
                return _NATIVE_NODE
    return _NO_NODE


def _without_node(tensors) -> bool:
    return _node_for(tensors) == _NO_NODE


def _forward(q, k, v, variant):
    status, out, lse = _host().attention_fwd(q, k, v, *variant, _stream(q))
    if status:
        fb.check(status)
    return out, lse


class _Attention(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, alibi_slopes, q_doc_ids, kv_doc_ids, variant):
        out, lse = _forward(q, k, v, variant)
        ctx.save_for_backward(q, k, v, out, lse)
        ctx.variant = variant
        return out

    @staticmethod
    def backward(ctx, dout):
        q, k, v, out, lse = ctx.saved_tensors
        status, dq, dk, dv = _host().attention_bwd(q, k, v, out, lse, dout, *ctx.variant, _stream(q))
        if status:
            fb.check(status)
        return dq, dk, dv, None, None, None, None


def attention(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, *, scale: Optional[float] = None,
              causal: bool = False, window: Optional[int] = None, prefix: Optional[int] = None,
              softcap: Optional[float] = None, alibi_slopes: Optional[torch.Tensor] = None,
              q_doc_ids: Optional[torch.Tensor] = None, kv_doc_ids: Optional[torch.Tensor] = None,
              q_offset: int = 0) -> torch.Tensor:
    """softmax(mask(score_mod(scale * q k^T))) v on the library's fused kernels, differentiable in
    q, k and v.  q [B, (G,) H, Sq, D], k and v [B, (G,) Hkv, Sk, D] with Hkv dividing H; bf16.

    alibi_slopes: float32 [H]; q_doc_ids / kv_doc_ids: int32 [B, Sq] / [B, Sk] (kv defaults to q's).
    q_offset: query row i sits at sequence position i + q_offset in the positional masks and ALiBi
    (Sk - Sq aligns a causal mask bottom-right: a chunk of new queries against a longer cache).
    """
    if not q.is_cuda or q.dtype != torch.bfloat16:
        raise ValueError("attention() takes bf16 CUDA tensors (there is no CPU or fallback path)")
    if scale is None:
        scale = q.shape[-1] ** -0.5
    if q_doc_ids is not None and kv_doc_ids is None:
        kv_doc_ids = q_doc_ids
    if kv_doc_ids is not None and q_doc_ids is None:
        raise ValueError("kv_doc_ids needs q_doc_ids")
    for x in (q, k, v):
        if x.dim() not in (4, 5):
            raise ValueError(f"expected [B, H, S, D] or [B, G, H, S, D], got {tuple(x.shape)}")
    if alibi_slopes is not None:
        _check_aux("alibi_slopes", alibi_slopes, torch.float32, (q.shape[-3],), q.device)
    if q_doc_ids is not None:
        _check_aux("q_doc_ids", q_doc_ids, torch.int32, (q.shape[0], q.shape[-2]), q.device)
        _check_aux("kv_doc_ids", kv_doc_ids, torch.int32, (k.shape[0], k.shape[-2]), q.device)
    if q_offset < 0:
        raise ValueError("q_offset must be >= 0")
    variant = (float(scale), _score_mod(softcap, alibi_slopes), float(softcap or 0.0), _mask_bits(causal, window, prefix, q_doc_ids),
               int(window or 0), int(prefix or 0), int(q_offset), alibi_slopes, q_doc_ids, kv_doc_ids)
    node = _node_for((q, k, v, alibi_slopes))
    if node == _NO_NODE:
        return _forward(q, k, v, variant)[0]
    if node == _NATIVE_NODE:
        status, out = _host().attention_node(q, k, v, *variant, _stream(q))
        if status:
            fb.check(status)
        return out
    return _Attention.apply(q, k, v, alibi_slopes, q_doc_ids, kv_doc_ids, variant)


def _variant_forward(tensors, variant):
    status, out, lse = _host().variant_fwd(*tensors, *variant, _stream(tensors[0]))
    if status:
        fb.check(status)
    return out, lse


class _VariantAttention(torch.autograd.Function):
    """Forward fl_attn_fwd, backward fl_attn_bwd_ex, for descriptors with biases / gate / RMSNorm / second stream.
    Tensor inputs: q, k, v, q2, k2, lam, gate, bias0, bias1, rms_weight (absent ones are None)."""

    @staticmethod
    def forward(ctx, variant, q, k, v, q2, k2, lam, gate, bias0, bias1, rms_weight):
        tensors = (q, k, v, q2, k2, lam, gate, bias0, bias1, rms_weight)
        out, lse = _variant_forward(tensors, variant)
        ctx.save_for_backward(*tensors, out, lse)
        ctx.variant = variant
        return out

    @staticmethod
    def backward(ctx, dout):
        saved = ctx.saved_tensors
        status, grads = _host().variant_bwd(*saved, dout, *ctx.variant, _stream(saved[0]))
        if status:
            fb.check(status)
        return (None, *grads)


def variant_attention(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, *, scale: Optional[float] = None,
                      causal: bool = False, window: Optional[int] = None, prefix: Optional[int] = None,
                      softcap: Optional[float] = None, alibi_slopes: Optional[torch.Tensor] = None,
                      q_doc_ids: Optional[torch.Tensor] = None, kv_doc_ids: Optional[torch.Tensor] = None,
                      q_offset: int = 0, biases=(), gate: Optional[torch.Tensor] = None,
                      q2: Optional[torch.Tensor] = None, k2: Optional[torch.Tensor] = None,
                      lam: Optional[torch.Tensor] = None, rmsnorm: bool = False, rms_eps: float = 1e-6,
                      rms_weight: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Every variant of the forward pass with autograd: attention() plus

    biases    up to two bf16 tensors that broadcast to [B, G, H, Sq, Sk] (5-D, size-1 axes broadcast), added to the
              scaled score; their gradients come back in the biases' own shapes
    gate      pre-sigmoid tensor of the output's shape: out = sigmoid(gate) * (...)
    q2, k2, lam   the second softmax stream of differential attention and its per-head fp32 weights [H]:
              softmax(q k^T) v - lam_h softmax(q2 k2^T) v
    rmsnorm   RMSNorm over the output channels (rms_weight fp32 [Dv] or None for all ones), before the gate
    Tensors are [B, H, S, D] or [B, G, H, S, D], bf16, on the GPU; differentiable in q, k, v, q2, k2, lam, gate, biases
    and rms_weight."""
    if not q.is_cuda or q.dtype != torch.bfloat16:
        raise ValueError("variant_attention() takes bf16 CUDA tensors (there is no CPU or fallback path)")
    if (q2 is None) != (k2 is None) or (q2 is None) != (lam is None):
        raise ValueError("q2, k2 and lam come together")
    if softcap is not None and alibi_slopes is not None:
        raise ValueError("one score_mod at a time")
    if len(biases) > 2:
        raise ValueError("at most two biases")
    q5, k5 = _as5(q), _as5(k)
    if q_doc_ids is not None and kv_doc_ids is None:
        kv_doc_ids = q_doc_ids
    _check_aux("alibi_slopes", alibi_slopes, torch.float32, (q5.shape[2],), q.device)
    _check_aux("q_doc_ids", q_doc_ids, torch.int32, (q5.shape[0], q5.shape[3]), q.device)
    _check_aux("kv_doc_ids", kv_doc_ids, torch.int32, (k5.shape[0], k5.shape[3]), q.device)
    _check_aux("lam", lam, torch.float32, (q5.shape[2],), q.device)
    if rms_weight is not None:
        _check_aux("rms_weight", rms_weight, torch.float32, (_as5(v).shape[4],), q.device)
    for n, b in enumerate(biases):
        if b.dim() != 5 or b.dtype != torch.bfloat16 or b.device != q.device:
            raise ValueError(f"biases[{n}] must be a 5-D bf16 tensor on {q.device}")
    variant = (float(q.shape[-1] ** -0.5 if scale is None else scale), _score_mod(softcap, alibi_slopes), float(softcap or 0.0),
               _mask_bits(causal, window, prefix, q_doc_ids), int(window or 0), int(prefix or 0), int(q_offset), bool(rmsnorm),
               float(rms_eps) if rmsnorm else 0.0, alibi_slopes, q_doc_ids, kv_doc_ids)
    b0 = biases[0] if len(biases) > 0 else None
    b1 = biases[1] if len(biases) > 1 else None
    tensors = (q, k, v, q2, k2, lam, gate, b0, b1, rms_weight if rmsnorm else None)
    node = _node_for(tensors)
    if node == _NO_NODE:
        return _variant_forward(tensors, variant)[0]
    if node == _NATIVE_NODE:
        status, out = _host().variant_node(*tensors, *variant, _stream(q))
        if status:
            fb.check(status)
        return out
    return _VariantAttention.apply(variant, *tensors)


def _paged_call(decode, q, k_cache, v_cache, seq_lens, block_table, max_seq_len, scale, window, softcap, alibi_slopes, workspace,
                return_lse):
    mask = (fb.FL_MASK_WINDOW | fb.FL_MASK_CAUSAL) if window is not None else fb.FL_MASK_CAUSAL
    status, need, out, lse = _host().paged(decode, q, k_cache, v_cache, seq_lens, block_table, int(max_seq_len), float(scale),
                                           _score_mod(softcap, alibi_slopes), float(softcap or 0.0), mask, int(window or 0),
                                           alibi_slopes, workspace, return_lse, _stream(q))
    if status:
        fb.check(status)
    if workspace is not None and workspace.numel() * workspace.element_size() < need:
        raise ValueError(f"workspace holds {workspace.numel() * workspace.element_size()} bytes, {need} needed")
    return (out, lse) if return_lse else out


def decode_attention(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, seq_lens: torch.Tensor,
                     block_table: Optional[torch.Tensor] = None, *, max_seq_len: Optional[int] = None,
                     scale: Optional[float] = None, window: Optional[int] = None, softcap: Optional[float] = None,
                     alibi_slopes: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                     return_lse: bool = False):
    """One decode step (fl_attn_decode): the last token of every sequence against its cached keys.

    q [B, H, D] bf16; k_cache, v_cache [pages, page_size, Hkv, D] bf16 (any strides with unit inner
    stride, e.g. a permuted [pages, Hkv, page_size, D] buffer); seq_lens int32 [B] on the device;
    block_table int32 [B, max_pages] or None for a contiguous cache (sequence b in "page" b).
    max_seq_len is a host-side bound on seq_lens (it fixes the launch shape; default: the capacity
    of the table, so no device value is read back).  workspace: a uint8 tensor of at least
    decode_workspace_size(...) bytes to reuse across steps; allocated here when omitted.
    Returns out [B, H, D] bf16 (and lse [B, H] float32 with return_lse).  Not differentiable.
    """
    if not q.is_cuda or q.dtype != torch.bfloat16 or q.dim() != 3:
        raise ValueError("decode_attention() takes a bf16 CUDA q of shape [B, H, D]")
    B, H, D = q.shape
    page_size = k_cache.shape[1]
    _check_aux("seq_lens", seq_lens, torch.int32, (B,), q.device)
    if block_table is not None:
        if block_table.dim() != 2:
            raise ValueError("block_table must be [B, max_pages]")
        _check_aux("block_table", block_table, torch.int32, (B, block_table.shape[1]), q.device, contiguous=False,
                   inner_unit=True)
    _check_aux("alibi_slopes", alibi_slopes, torch.float32, (H,), q.device)
    if max_seq_len is None:
        max_seq_len = (block_table.shape[1] if block_table is not None else 1) * page_size
    if scale is None:
        scale = D ** -0.5
    return _paged_call(True, q, k_cache, v_cache, seq_lens, block_table, max_seq_len, scale, window, softcap, alibi_slopes, workspace,
                       return_lse)


def paged_prefill_attention(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, seq_lens: torch.Tensor,
                            block_table: Optional[torch.Tensor] = None, *, max_seq_len: Optional[int] = None,
                            scale: Optional[float] = None, window: Optional[int] = None, softcap: Optional[float] = None,
                            alibi_slopes: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                            return_lse: bool = False):
    """A chunk of query rows per sequence against the paged cache (fl_attn_prefill_paged): the last Sq tokens of every
    sequence, whose keys and values are already cached, attend causally to that sequence's cached keys.

    q [B, H, Sq, D] bf16; caches, seq_lens, block_table, max_seq_len as for decode_attention().  workspace: a uint8
    tensor of at least prefill workspace bytes (two dense copies of the cached rows) to reuse across calls;
    allocated here when omitted.  Returns out [B, H, Sq, D] bf16 (and lse [B, H, Sq] float32 with return_lse);
    rows at negative positions (a sequence shorter than the chunk) are zero.  Not differentiable."""
    if not q.is_cuda or q.dtype != torch.bfloat16 or q.dim() != 4:
        raise ValueError("paged_prefill_attention() takes a bf16 CUDA q of shape [B, H, Sq, D]")
    B, H, Sq, D = q.shape
    page_size = k_cache.shape[1]
    _check_aux("seq_lens", seq_lens, torch.int32, (B,), q.device)
    if block_table is not None:
        if block_table.dim() != 2:
            raise ValueError("block_table must be [B, max_pages]")
        _check_aux("block_table", block_table, torch.int32, (B, block_table.shape[1]), q.device, contiguous=False,
                   inner_unit=True)
    _check_aux("alibi_slopes", alibi_slopes, torch.float32, (H,), q.device)
    if max_seq_len is None:
        max_seq_len = (block_table.shape[1] if block_table is not None else 1) * page_size
    if scale is None:
        scale = D ** -0.5
    return _paged_call(False, q, k_cache, v_cache, seq_lens, block_table, max_seq_len, scale, window, softcap, alibi_slopes, workspace,
                       return_lse)
