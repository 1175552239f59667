// Marshalling of the PyTorch entry points (attention and its backward pass, with and without the variants' extra tensors, a decode
// step, a chunk of a paged prefill): torch tensors in, C-ABI descriptors filled, outputs and workspace taken from torch's
// allocator, one call of libflattn.so, the fl_status and the outputs back.  No attention arithmetic and no kernel is here.
//
// The same in Python (ctypes structures filled field by field) cost 20 us of a 31 us causal call on [1, 8, 128, 64] and of
// a 31 us decode step of one sequence, whose kernels take 8 and 10 us; a training step with a bias and a gate on
// [1, 16, 4, 64, 32] took 252 us that way and 117 this way with autograd nodes in Python, most of it in the autograd engine.
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/extension.h>

#include <optional>
#include <tuple>

#include "../../include/fl_attn.h"

namespace py = pybind11;
using at::Tensor;
typedef std::optional<Tensor> OptTensor;

namespace {

int dtype_code(const Tensor& t) {
  switch (t.scalar_type()) {
    case at::kBFloat16: return FL_BF16;
    case at::kFloat: return FL_F32;
    case at::kInt: return FL_I32;
    default: throw py::key_error(c10::toString(t.scalar_type()));
  }
}

// The 5-D descriptor of a tensor whose axes are `axes` (-1: an axis of size 1).
fl_tensor desc5(const Tensor& t, const int (&axes)[5]) {
  fl_tensor d = {};
  d.ptr = t.data_ptr();
  d.dtype = dtype_code(t);
  for (int a = 0; a < 5; ++a) {
    d.size[a] = axes[a] < 0 ? 1 : t.size(axes[a]);
    d.stride[a] = axes[a] < 0 ? 0 : t.stride(axes[a]);
  }
  return d;
}
// [B, H, S, D] or [B, G, H, S, D]
fl_tensor desc(const Tensor& t) {
  if (t.dim() == 5) return desc5(t, {0, 1, 2, 3, 4});
  if (t.dim() != 4) throw py::value_error("expected [B, H, S, D] or [B, G, H, S, D], got " + std::to_string(t.dim()) + " axes");
  return desc5(t, {0, -1, 1, 2, 3});
}

template <class T>
T* ptr(const OptTensor& t) {
  return t.has_value() ? (T*)t->data_ptr() : nullptr;
}

fl_variant_desc variant(double scale, int mod, double softcap, int mask, int window, int prefix, int q_offset) {
  fl_variant_desc d = {};
  d.struct_size = sizeof(d);
  d.scale = (float)scale;
  d.score_mod = (uint32_t)mod;
  d.softcap = (float)softcap;
  d.mask = (uint32_t)mask;
  d.window = window;
  d.prefix_len = prefix;
  d.q_offset = q_offset;
  return d;
}

fl_aux aux_of(const OptTensor& slopes, const OptTensor& q_ids, const OptTensor& kv_ids, const Tensor& workspace) {
  fl_aux a = {};
  a.struct_size = sizeof(a);
  a.alibi_slopes = ptr<const float>(slopes);
  a.q_doc_ids = ptr<const int32_t>(q_ids);
  a.kv_doc_ids = ptr<const int32_t>(kv_ids);
  if (workspace.defined()) {
    a.workspace = workspace.data_ptr();
    a.workspace_bytes = workspace.nbytes();
  }
  return a;
}

// An output gradient in a layout that the kernels read: unit inner stride, 16-byte aligned rows and base, no broadcast axis
// (autograd hands over a sum over an outer axis as one).
Tensor readable(const Tensor& t) {
  bool ok = t.stride(-1) == 1 && (uintptr_t)t.data_ptr() % 16 == 0;
  for (int64_t a = 0; a + 1 < t.dim(); ++a) ok = ok && (t.size(a) == 1 || (t.stride(a) != 0 && t.stride(a) % 8 == 0));
  return ok ? t : t.clone(at::MemoryFormat::Contiguous);
}

Tensor bytes(size_t n, const Tensor& like) { return at::empty({(int64_t)n}, like.options().dtype(at::kByte)); }

// out [B, (G,) H, Sq, Dv] in q's dtype and rank, lse [B, G, H, Sq, 1]
std::tuple<int, Tensor, Tensor> attention_fwd(const Tensor& q, const Tensor& k, const Tensor& v, double scale, int mod, double softcap,
                                              int mask, int window, int prefix, int q_offset, const OptTensor& slopes,
                                              const OptTensor& q_ids, const OptTensor& kv_ids, int64_t stream) {
  const fl_tensor tq = desc(q), tk = desc(k), tv = desc(v);
  const fl_variant_desc d = variant(scale, mod, softcap, mask, window, prefix, q_offset);
  std::vector<int64_t> size(q.sizes().begin(), q.sizes().end());
  size.back() = tv.size[4];
  Tensor out = at::empty(size, q.options());
  Tensor lse = at::empty({tq.size[0], tq.size[1], tq.size[2], tq.size[3], 1}, q.options().dtype(at::kFloat));
  fl_tensor tout = desc(out), tlse = desc(lse);
  Tensor ws;
  const size_t need = fl_attn_fwd_workspace_size(&tq, &tk, &d);
  if (need != 0) ws = bytes(need, q);
  const fl_aux a = aux_of(slopes, q_ids, kv_ids, ws);
  const int status = fl_attn_fwd(&tq, &tk, &tv, &d, &a, &tout, &tlse, (void*)stream);
  return {status, out, lse};
}

// dq, dk, dv in the layouts of q, k, v
std::tuple<int, Tensor, Tensor, Tensor> attention_bwd(const Tensor& q, const Tensor& k, const Tensor& v, const Tensor& out,
                                                      const Tensor& lse, const Tensor& dout_in, double scale, int mod, double softcap,
                                                      int mask, int window, int prefix, int q_offset, const OptTensor& slopes,
                                                      const OptTensor& q_ids, const OptTensor& kv_ids, int64_t stream) {
  const Tensor dout = readable(dout_in);
  const fl_tensor tq = desc(q), tk = desc(k), tv = desc(v), tout = desc(out), tlse = desc(lse), tdo = desc(dout);
  const fl_variant_desc d = variant(scale, mod, softcap, mask, window, prefix, q_offset);
  Tensor dq = at::empty_like(q), dk = at::empty_like(k), dv = at::empty_like(v);
  fl_tensor tdq = desc(dq), tdk = desc(dk), tdv = desc(dv);
  const Tensor ws = bytes(std::max<size_t>(fl_attn_bwd_workspace_size(&tq, &tk, &d), 16), q);
  const fl_aux a = aux_of(slopes, q_ids, kv_ids, ws);
  const int status = fl_attn_bwd(&tq, &tk, &tv, &tout, &tdo, &tlse, &d, &a, &tdq, &tdk, &tdv, (void*)stream);
  return {status, dq, dk, dv};
}

// The tensors of a variant beyond q, k and v (absent ones are None), as variant_fwd and variant_bwd take them.
struct Extras {
  const OptTensor &q2, &k2, &lam, &gate, &bias0, &bias1, &rms_weight;
  int n_bias() const { return (int)bias0.has_value() + (int)bias1.has_value(); }
  fl_variant_desc describe(fl_variant_desc d, bool rmsnorm, double rms_eps) const {
    d.n_bias = (uint32_t)n_bias();
    d.combine = q2.has_value() ? FL_DIFFERENTIAL : FL_SINGLE;
    d.epilogue = (rmsnorm ? FL_EPI_RMSNORM : 0) | (gate.has_value() ? FL_EPI_GATE_SIGMOID : 0);
    d.rms_eps = rmsnorm ? (float)rms_eps : 0.f;
    return d;
  }
  fl_aux fill(fl_aux a) const {
    int n = 0;
    for (const OptTensor* b : {&bias0, &bias1})
      if (b->has_value()) a.bias[n++] = desc(**b);
    if (gate.has_value()) a.gate = desc(*gate);
    if (q2.has_value()) a.q2 = desc(*q2);
    if (k2.has_value()) a.k2 = desc(*k2);
    a.lambda = ptr<const float>(lam);
    a.rms_weight = ptr<const float>(rms_weight);
    return a;
  }
};

// out in q's dtype and rank, lse [B, G or 2 G (two streams), H, Sq, 1]
std::tuple<int, Tensor, Tensor> variant_fwd(const Tensor& q, const Tensor& k, const Tensor& v, const OptTensor& q2, const OptTensor& k2,
                                            const OptTensor& lam, const OptTensor& gate, const OptTensor& bias0, const OptTensor& bias1,
                                            const OptTensor& rms_weight, double scale, int mod, double softcap, int mask, int window,
                                            int prefix, int q_offset, bool rmsnorm, double rms_eps, const OptTensor& slopes,
                                            const OptTensor& q_ids, const OptTensor& kv_ids, int64_t stream) {
  const Extras x{q2, k2, lam, gate, bias0, bias1, rms_weight};
  const fl_tensor tq = desc(q), tk = desc(k), tv = desc(v);
  const fl_variant_desc d = x.describe(variant(scale, mod, softcap, mask, window, prefix, q_offset), rmsnorm, rms_eps);
  std::vector<int64_t> size(q.sizes().begin(), q.sizes().end());
  size.back() = tv.size[4];
  Tensor out = at::empty(size, q.options());
  Tensor lse = at::empty({tq.size[0], (q2.has_value() ? 2 : 1) * tq.size[1], tq.size[2], tq.size[3], 1}, q.options().dtype(at::kFloat));
  fl_tensor tout = desc(out), tlse = desc(lse);
  Tensor ws;
  const size_t need = fl_attn_fwd_workspace_size(&tq, &tk, &d);
  if (need != 0) ws = bytes(need, q);
  const fl_aux a = x.fill(aux_of(slopes, q_ids, kv_ids, ws));
  const int status = fl_attn_fwd(&tq, &tk, &tv, &d, &a, &tout, &tlse, (void*)stream);
  return {status, out, lse};
}

// The status and the gradients of q, k, v, q2, k2, lam, gate, bias0, bias1, rms_weight in their layouts (None where absent).  The
// kernels sum bias gradients in fp32; they are rounded to the biases' dtype here.
std::tuple<int, std::vector<OptTensor>> variant_bwd(const Tensor& q, const Tensor& k, const Tensor& v, const OptTensor& q2,
                                                    const OptTensor& k2, const OptTensor& lam, const OptTensor& gate,
                                                    const OptTensor& bias0, const OptTensor& bias1, const OptTensor& rms_weight,
                                                    const Tensor& out, const Tensor& lse, const Tensor& dout_in, double scale, int mod,
                                                    double softcap, int mask, int window, int prefix, int q_offset, bool rmsnorm,
                                                    double rms_eps, const OptTensor& slopes, const OptTensor& q_ids,
                                                    const OptTensor& kv_ids, int64_t stream) {
  const Extras x{q2, k2, lam, gate, bias0, bias1, rms_weight};
  const Tensor dout = readable(dout_in);
  const fl_tensor tq = desc(q), tk = desc(k), tv = desc(v), tout = desc(out), tlse = desc(lse), tdo = desc(dout);
  const fl_variant_desc d = x.describe(variant(scale, mod, softcap, mask, window, prefix, q_offset), rmsnorm, rms_eps);
  auto like = [](const OptTensor& t) { return t.has_value() ? OptTensor(at::empty_like(*t)) : OptTensor(); };
  auto fp32 = [](const OptTensor& t) { return t.has_value() ? OptTensor(at::empty(t->sizes(), t->options().dtype(at::kFloat))) : OptTensor(); };
  Tensor dq = at::empty_like(q), dk = at::empty_like(k), dv = at::empty_like(v);
  const OptTensor dq2 = like(q2), dk2 = like(k2), dlam = like(lam), dgate = like(gate), drms = fp32(rms_weight);
  OptTensor dbias0 = fp32(bias0), dbias1 = fp32(bias1);
  fl_bwd_extra e = {};
  e.struct_size = sizeof(e);
  if (dq2.has_value()) e.dq2 = desc(*dq2);
  if (dk2.has_value()) e.dk2 = desc(*dk2);
  if (dgate.has_value()) e.dgate = desc(*dgate);
  int n = 0;
  for (const OptTensor* b : {&dbias0, &dbias1})
    if (b->has_value()) e.dbias[n++] = desc(**b);
  e.dlambda = ptr<float>(dlam);
  e.drms_weight = ptr<float>(drms);
  fl_tensor tdq = desc(dq), tdk = desc(dk), tdv = desc(dv);
  const Tensor ws = bytes(std::max<size_t>(fl_attn_bwd_ex_workspace_size(&tq, &tk, &tv, &d), 16), q);
  const fl_aux a = x.fill(aux_of(slopes, q_ids, kv_ids, ws));
  const int status = fl_attn_bwd_ex(&tq, &tk, &tv, &tout, &tdo, &tlse, &d, &a, &tdq, &tdk, &tdv, &e, (void*)stream);
  if (status == 0) {
    if (dbias0.has_value()) dbias0 = dbias0->to(bias0->scalar_type());
    if (dbias1.has_value()) dbias1 = dbias1->to(bias1->scalar_type());
  }
  return {status, {dq, dk, dv, dq2, dk2, dlam, dgate, dbias0, dbias1, drms}};
}

// A decode step (q [B, H, D]) or a chunk of a paged prefill (q [B, H, Sq, D]) over caches [pages, page_size, Hkv, D].  Returns
// the status, the workspace bytes the call needs, out (q's shape) and lse ([B, H] or [B, H, Sq]; undefined unless wanted).  A
// workspace that is too small is reported by the second value alone: nothing has been launched then.
std::tuple<int, int64_t, Tensor, OptTensor> paged(bool decode, const Tensor& q, const Tensor& k_cache, const Tensor& v_cache,
                                                  const Tensor& seq_lens, const OptTensor& table, int max_seq_len, double scale,
                                                  int mod, double softcap, int mask, int window, const OptTensor& slopes,
                                                  const OptTensor& workspace, bool want_lse, int64_t stream) {
  TORCH_CHECK(k_cache.dim() == 4 && v_cache.dim() == 4, "the caches must be [pages, page_size, Hkv, D]");
  const fl_tensor tq = decode ? desc5(q, {0, -1, 1, -1, 2}) : desc5(q, {0, -1, 1, 2, 3});
  const fl_tensor tk = desc5(k_cache, {0, -1, 2, 1, 3}), tv = desc5(v_cache, {0, -1, 2, 1, 3});
  Tensor out = at::empty(q.sizes(), q.options());
  fl_tensor tout = decode ? desc5(out, {0, -1, 1, -1, 2}) : desc5(out, {0, -1, 1, 2, 3});
  OptTensor lse;
  fl_tensor tlse = {};
  if (want_lse) {
    lse = at::empty(q.sizes().slice(0, q.dim() - 1), q.options().dtype(at::kFloat));
    tlse = decode ? desc5(*lse, {0, -1, 1, -1, -1}) : desc5(*lse, {0, -1, 1, 2, -1});
  }
  fl_paged_kv kv = {};
  kv.struct_size = sizeof(kv);
  kv.block_table = ptr<const int32_t>(table);
  kv.table_stride = table.has_value() ? (int32_t)table->stride(0) : 0;
  kv.page_size = (int32_t)k_cache.size(1);
  kv.seq_lens = (const int32_t*)seq_lens.data_ptr();
  kv.max_seq_len = max_seq_len;
  const size_t need = std::max<size_t>(
      decode ? fl_attn_decode_workspace_size(&tq, &tk, &kv) : fl_attn_prefill_paged_workspace_size(&tq, &tk, &kv), 16);
  if (workspace.has_value() && workspace->nbytes() < need) return {0, (int64_t)need, out, lse};
  const Tensor ws = workspace.has_value() ? *workspace : bytes(need, q);
  const fl_variant_desc d = variant(scale, mod, softcap, mask, window, 0, 0);
  const fl_aux a = aux_of(slopes, std::nullopt, std::nullopt, ws);
  const int status = (decode ? fl_attn_decode : fl_attn_prefill_paged)(&tq, &tk, &tv, &kv, &d, &a, &tout, want_lse ? &tlse : nullptr,
                                                                      (void*)stream);
  return {status, (int64_t)need, out, lse};
}

// ---- the autograd nodes of training calls.  A node written in Python is entered by the engine's thread under the interpreter's lock, which
// the calling thread has just given up.  A causal forward and backward call on [1, 8, 110, 128] took 45 or 89 us with one, by where the
// process runs, and takes 38 or 72 with these; documents and windows 3 x 32/8 x 182 61 or 97, and 49 or 84.  Calls under a transform, a
// trace, forward-mode derivatives or torch.compile keep the Python node (functional.py).

PyObject* g_check = nullptr;                       // binding.check: raises for a status

// The exception that binding.check raises for `status`, thrown on a thread without the interpreter's lock; the engine carries it to the caller.
[[noreturn]] void throw_status(int status) {
  py::gil_scoped_acquire gil;
  PyObject* r = PyObject_CallFunction(g_check, "i", status);
  if (r != nullptr) {                              // (not reached: it raises for every status but 0)
    Py_DECREF(r);
    PyErr_SetString(PyExc_RuntimeError, "backward pass failed");
  }
  python_error e;
  e.persist();
  throw e;
}

int64_t current_stream(const Tensor& t) { return (int64_t)c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

// The outputs of a forward pass, taken through Function::apply unseen, and what its backward pass needs beside tensors that autograd saves.
struct Done {
  const Tensor &out, &lse;
  const std::vector<double>& scalars;
  const OptTensor &slopes, &q_ids, &kv_ids;

  void keep(torch::autograd::AutogradContext* ctx) const {
    ctx->saved_data["scalars"] = scalars;
    if (slopes.has_value()) ctx->saved_data["slopes"] = *slopes;
    if (q_ids.has_value()) ctx->saved_data["q_ids"] = *q_ids;
    if (kv_ids.has_value()) ctx->saved_data["kv_ids"] = *kv_ids;
  }
};
OptTensor kept(torch::autograd::AutogradContext* ctx, const char* name) {
  const auto it = ctx->saved_data.find(name);
  return it == ctx->saved_data.end() ? OptTensor() : OptTensor(it->second.toTensor());
}
// (slopes are an input without a gradient: a call that only they would need a derivative of has a node all the same)
struct AttentionNode : torch::autograd::Function<AttentionNode> {
  static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& q, const Tensor& k, const Tensor& v, const OptTensor&, const Done& done) {
    ctx->save_for_backward({q, k, v, done.out, done.lse});
    done.keep(ctx);
    return done.out;
  }
  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, const torch::autograd::variable_list& grads) {
    const auto t = ctx->get_saved_variables();
    const auto s = ctx->saved_data["scalars"].toDoubleVector();
    auto [status, dq, dk, dv] = attention_bwd(t[0], t[1], t[2], t[3], t[4], grads[0], s[0], (int)s[1], s[2], (int)s[3], (int)s[4], (int)s[5],
                                              (int)s[6], kept(ctx, "slopes"), kept(ctx, "q_ids"), kept(ctx, "kv_ids"), current_stream(t[0]));
    if (status != 0) throw_status(status);
    return {dq, dk, dv, Tensor(), Tensor()};
  }
};

// attention_fwd with a node: the status and out
std::tuple<int, Tensor> attention_node(const Tensor& q, const Tensor& k, const Tensor& v, double scale, int mod, double softcap, int mask,
                                       int window, int prefix, int q_offset, const OptTensor& slopes, const OptTensor& q_ids,
                                       const OptTensor& kv_ids, int64_t stream) {
  auto [status, out, lse] = attention_fwd(q, k, v, scale, mod, softcap, mask, window, prefix, q_offset, slopes, q_ids, kv_ids, stream);
  if (status != 0) return {status, out};
  const std::vector<double> scalars = {scale, (double)mod, softcap, (double)mask, (double)window, (double)prefix, (double)q_offset};
  return {0, AttentionNode::apply(q, k, v, slopes, Done{out, lse, scalars, slopes, q_ids, kv_ids})};
}

struct VariantNode : torch::autograd::Function<VariantNode> {
  static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& q, const Tensor& k, const Tensor& v, const OptTensor& q2,
                        const OptTensor& k2, const OptTensor& lam, const OptTensor& gate, const OptTensor& bias0, const OptTensor& bias1,
                        const OptTensor& rms_weight, const Done& done) {
    torch::autograd::variable_list saved = {q, k, v};
    for (const OptTensor* x : {&q2, &k2, &lam, &gate, &bias0, &bias1, &rms_weight}) saved.push_back(x->has_value() ? **x : Tensor());
    saved.push_back(done.out);
    saved.push_back(done.lse);
    ctx->save_for_backward(std::move(saved));
    done.keep(ctx);
    return done.out;
  }
  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, const torch::autograd::variable_list& grads) {
    const auto t = ctx->get_saved_variables();
    const auto s = ctx->saved_data["scalars"].toDoubleVector();
    auto opt = [](const Tensor& x) { return x.defined() ? OptTensor(x) : OptTensor(); };
    auto [status, g] = variant_bwd(t[0], t[1], t[2], opt(t[3]), opt(t[4]), opt(t[5]), opt(t[6]), opt(t[7]), opt(t[8]), opt(t[9]), t[10], t[11],
                                   grads[0], s[0], (int)s[1], s[2], (int)s[3], (int)s[4], (int)s[5], (int)s[6], s[7] != 0, s[8], kept(ctx, "slopes"),
                                   kept(ctx, "q_ids"), kept(ctx, "kv_ids"), current_stream(t[0]));
    if (status != 0) throw_status(status);
    torch::autograd::variable_list out;
    for (const OptTensor& x : g) out.push_back(x.has_value() ? *x : Tensor());
    out.emplace_back();                            // the forward pass's results
    return out;
  }
};

// variant_fwd with a node: the status and out
std::tuple<int, Tensor> variant_node(const Tensor& q, const Tensor& k, const Tensor& v, const OptTensor& q2, const OptTensor& k2, const OptTensor& lam,
                                     const OptTensor& gate, const OptTensor& bias0, const OptTensor& bias1, const OptTensor& rms_weight,
                                     double scale, int mod, double softcap, int mask, int window, int prefix, int q_offset, bool rmsnorm,
                                     double rms_eps, const OptTensor& slopes, const OptTensor& q_ids, const OptTensor& kv_ids, int64_t stream) {
  auto [status, out, lse] = variant_fwd(q, k, v, q2, k2, lam, gate, bias0, bias1, rms_weight, scale, mod, softcap, mask, window, prefix, q_offset,
                                        rmsnorm, rms_eps, slopes, q_ids, kv_ids, stream);
  if (status != 0) return {status, out};
  const std::vector<double> scalars = {scale,          (double)mod,      softcap, (double)mask, (double)window,
                                       (double)prefix, (double)q_offset, rmsnorm ? 1.0 : 0.0, rms_eps};
  return {0, VariantNode::apply(q, k, v, q2, k2, lam, gate, bias0, bias1, rms_weight, Done{out, lse, scalars, slopes, q_ids, kv_ids})};
}

}  // namespace

PYBIND11_MODULE(_fltorch, m) {
  typedef py::call_guard<py::gil_scoped_release> nogil;
  m.def("attention_fwd", &attention_fwd, nogil());
  m.def("attention_bwd", &attention_bwd, nogil());
  m.def("attention_node", &attention_node, nogil());
  m.def("variant_fwd", &variant_fwd, nogil());
  m.def("variant_bwd", &variant_bwd, nogil());
  m.def("variant_node", &variant_node, nogil());
  m.def("paged", &paged, nogil());
  m.def("set_check", [](py::object check) {
    Py_XDECREF(g_check);
    g_check = check.release().ptr();
  });
}
