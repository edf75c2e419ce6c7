// The calls of ops.py that sit on a user's path, marshalled in native code: the
// argument checks, the allocations and the library call of the forward entry
// points, and the autograd node of mra_attention. The library itself is bound
// at run time (bind: the addresses of the C ABI of the libmra.so that ops.load
// opened), so there is one copy of it in the process.
//
// Why native: at small sizes a call is its host time. One sequence of 512 tokens
// x 12 heads (forward and backward, seven launches, 48 us on the GPU) took 184 us
// a step with the Python autograd function, 41 of them in the forward and the
// rest mostly on the autograd engine's thread; with this node it takes 58 in a
// bare loop and 91 among other work. A forward call's host time fell from 19 to
// 12 us, which is its three launches.
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>

#include "mra.h"

namespace py = pybind11;

namespace {

constexpr int kBlock = 32;

// the library's entry points used here
struct Api {
  decltype(&mra_forward_workspace_bytes) forward_ws;
  decltype(&mra_attention_forward) forward;
  decltype(&mra_sparse_attention_forward) sparse;
  decltype(&mra_forward_global_workspace_bytes) global_ws;
  decltype(&mra_attention_forward_global) global;
  decltype(&mra_forward_pooled_rows) pooled_rows;
  decltype(&mra_backward_workspace_bytes) backward_ws;
  decltype(&mra_attention_backward) backward;
  decltype(&mra_attention_backward_pooled) backward_pooled;
};
Api api{};

enum Variant { kMra2 = 0, kSparse = 1, kGlobal = 2 };

// ops.py's MraError factory; never destroyed (the interpreter ends first)
py::object& status_error = *new py::object();

// What fails here is raised as the Python function of ops.py raises it, also from
// the backward, whose errors reach the caller through the autograd engine: a
// refusal by the library as MraError, one by the checks as c10's ValueError and
// TypeError, which torch turns into Python's (as it does its own, an exhausted
// allocator's, and a saved-tensor hook's exception).
void ok(const char* fn, mra_status_t st) {
  if (st == MRA_OK) return;
  py::gil_scoped_acquire gil;
  const py::object err = status_error(fn, (int)st);
  PyErr_SetObject(reinterpret_cast<PyObject*>(Py_TYPE(err.ptr())), err.ptr());
  python_error e;
  e.persist();
  throw e;
}

mra_dtype_t dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return MRA_F32;
  if (t.scalar_type() == at::kBFloat16) return MRA_BF16;
  TORCH_CHECK_TYPE(false, "unsupported dtype ", c10::toString(t.scalar_type()), "; expected float32 or bfloat16");
}

void check_like(const at::Tensor& t, const at::Tensor& ref) {
  TORCH_CHECK_VALUE(t.is_cuda(), "tensors must be on a ROCm device");
  TORCH_CHECK_VALUE(t.dim() == 4 && t.sizes() == ref.sizes() && t.scalar_type() == ref.scalar_type() &&
                        t.device() == ref.device(),
                    "q, k, v must share shape [B, H, n, d], dtype and device");
  TORCH_CHECK_VALUE(t.is_contiguous(), "q, k, v must be contiguous");
}

// A shape as Python writes it.
std::string tuple_of(at::IntArrayRef shape) {
  std::string s = "(";
  for (size_t i = 0; i < shape.size(); ++i) s += (i ? ", " : "") + std::to_string(shape[i]);
  return s + (shape.size() == 1 ? ",)" : ")");
}

void check_f32(const at::Tensor& t, at::IntArrayRef shape, const char* name) {
  TORCH_CHECK_VALUE(t.scalar_type() == at::kFloat && t.sizes() == shape && t.is_contiguous() && t.is_cuda(), name,
                    " must be a contiguous float32 device tensor of shape ", tuple_of(shape));
}

void check_idx(const at::Tensor& t, at::IntArrayRef shape, const at::Device& dev) {
  TORCH_CHECK_VALUE(t.scalar_type() == at::kInt && t.sizes() == shape && t.is_contiguous() && t.device() == dev,
                    "idx must be a contiguous int32 tensor of shape ", tuple_of(shape));
}

void* ptr(const std::optional<at::Tensor>& t) { return t ? t->data_ptr() : nullptr; }

struct Dims {
  int B, H, n, d;
};
Dims dims(const at::Tensor& t) { return {(int)t.size(0), (int)t.size(1), (int)t.size(2), (int)t.size(3)}; }

void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

size_t workspace_bytes(int variant, const Dims& s, int64_t budget, mra_dtype_t dt) {
  return variant == kGlobal ? api.global_ws(s.B, s.H, s.n, s.d, kBlock, dt)
                            : api.forward_ws(s.B, s.H, s.n, s.d, kBlock, (int)budget, dt);
}

void call_forward(int variant, const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const at::Tensor& out,
                  int32_t* idx, float* lse, void* ws, size_t ws_bytes, const Dims& s, int64_t budget, bool prior,
                  mra_dtype_t dt) {
  void* st = stream_of(q);
  const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
  void* o = out.data_ptr();
  if (variant == kGlobal)
    ok("mra_attention_forward_global",
       api.global(qp, kp, vp, o, idx, lse, ws, ws_bytes, s.B, s.H, s.n, s.d, kBlock, (int)budget, prior, dt, st));
  else if (variant == kSparse)
    ok("mra_sparse_attention_forward",
       api.sparse(qp, kp, vp, o, idx, lse, ws, ws_bytes, s.B, s.H, s.n, s.d, kBlock, (int)budget, dt, st));
  else
    ok("mra_attention_forward",
       api.forward(qp, kp, vp, o, idx, lse, ws, ws_bytes, s.B, s.H, s.n, s.d, kBlock, (int)budget, dt, st));
}

// One forward call: ops.attention_forward, sparse_attention_forward and
// attention_forward_global.
at::Tensor forward(int variant, const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, int64_t budget,
                   bool prior, std::optional<at::Tensor> out, const std::optional<at::Tensor>& idx_out,
                   const std::optional<at::Tensor>& workspace, const std::optional<at::Tensor>& lse_out) {
  for (const at::Tensor* t : {&q, &k, &v}) check_like(*t, q);
  const Dims s = dims(q);
  const int nb = s.n / kBlock;
  if (!out) out = at::empty_like(q);
  if (idx_out) check_idx(*idx_out, {s.B, s.H, nb, variant == kGlobal ? nb : budget}, q.device());
  if (lse_out) check_f32(*lse_out, {s.B, s.H, s.n}, "lse_out");
  const mra_dtype_t dt = dtype_code(q);
  at::Tensor ws;
  if (workspace) {
    ws = *workspace;
  } else {
    const size_t need = workspace_bytes(variant, s, budget, dt);
    ws = at::empty({(int64_t)(need ? need : 1)}, q.options().dtype(at::kByte));
  }
  call_forward(variant, q, k, v, *out, static_cast<int32_t*>(ptr(idx_out)), static_cast<float*>(ptr(lse_out)),
               ws.data_ptr(), ws.nbytes(), s, budget, prior, dt);
  return *out;
}

// The gradients (ops.attention_backward with everything allocated here).
// pooled: three block means or none.
std::vector<at::Tensor> backward(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const at::Tensor& out,
                                 const at::Tensor& dout, const at::Tensor& lse, const at::Tensor& idx, bool coarse,
                                 at::ArrayRef<at::Tensor> pooled) {
  for (const at::Tensor* t : {&q, &k, &v, &out, &dout}) check_like(*t, q);
  const Dims s = dims(q);
  const int nb = s.n / kBlock, width = (int)idx.size(-1);
  check_idx(idx, {s.B, s.H, nb, width}, q.device());
  check_f32(lse, {s.B, s.H, s.n}, "lse");
  const mra_dtype_t dt = dtype_code(q);
  at::Tensor dq = at::empty_like(q), dk = at::empty_like(q), dv = at::empty_like(q);
  const size_t need = api.backward_ws(s.B, s.H, s.n, s.d, kBlock, dt);
  at::Tensor ws = at::empty({(int64_t)(need ? need : 1)}, q.options().dtype(at::kByte));
  const float* lp = static_cast<const float*>(lse.data_ptr());
  const int32_t* ip = static_cast<const int32_t*>(idx.data_ptr());
  if (pooled.empty()) {
    ok("mra_attention_backward",
       api.backward(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), dout.data_ptr(), lp, ip, dq.data_ptr(),
                    dk.data_ptr(), dv.data_ptr(), ws.data_ptr(), ws.nbytes(), s.B, s.H, s.n, s.d, kBlock, width, coarse,
                    dt, stream_of(q)));
  } else {
    const char* names[3] = {"qp", "kp", "vp"};
    for (int i = 0; i < 3; ++i) {
      check_f32(pooled[i], {s.B, s.H, nb, s.d}, names[i]);
      TORCH_CHECK_VALUE(pooled[i].device() == q.device(), names[i], " must be on ", q.device());
    }
    ok("mra_attention_backward_pooled",
       api.backward_pooled(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), dout.data_ptr(), lp, ip,
                           static_cast<const float*>(pooled[0].data_ptr()), static_cast<const float*>(pooled[1].data_ptr()),
                           static_cast<const float*>(pooled[2].data_ptr()), dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
                           ws.data_ptr(), ws.nbytes(), s.B, s.H, s.n, s.d, kBlock, width, coarse, dt, stream_of(q)));
  }
  return {dq, dk, dv};
}

// ops.mra_attention: the node keeps its selection, log normalisers and block
// means as saved tensors (hooks on saved tensors see each of them).
struct Attention : torch::autograd::Function<Attention> {
  static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& q, const at::Tensor& k,
                            const at::Tensor& v, int64_t budget, int64_t variant, bool prior) {
    for (const at::Tensor* t : {&q, &k, &v}) check_like(*t, q);
    const Dims s = dims(q);
    const int nb = s.n / kBlock;
    const auto f32 = q.options().dtype(at::kFloat);
    at::Tensor lse = at::empty({s.B, s.H, s.n}, f32);
    at::Tensor idx = at::empty({s.B, s.H, nb, variant == kGlobal ? nb : budget}, q.options().dtype(at::kInt));
    const mra_dtype_t dt = dtype_code(q);
    const size_t need = workspace_bytes((int)variant, s, budget, dt);   // whole floats
    at::Tensor ws = at::empty({(int64_t)(need ? need / 4 : 1)}, f32);
    at::Tensor out = at::empty_like(q);
    call_forward((int)variant, q, k, v, out, idx.data_ptr<int32_t>(), lse.data_ptr<float>(), ws.data_ptr(), ws.nbytes(), s,
                 budget, prior, dt);
    std::vector<at::Tensor> save = {q, k, v, out, lse, idx};
    if (variant != kSparse) {
      const int64_t size = (int64_t)s.B * s.H * nb * s.d;
      const float* p[3] = {nullptr, nullptr, nullptr};
      if (size > 0)
        ok("mra_forward_pooled_rows",
           api.pooled_rows(ws.data_ptr(), s.B, s.H, s.n, s.d, kBlock, &p[0], &p[1], &p[2]));
      for (const float* x : p)
        save.push_back(size > 0 ? ws.narrow(0, x - ws.data_ptr<float>(), size).view({s.B, s.H, nb, s.d})
                                : at::empty({s.B, s.H, nb, s.d}, f32));
    }
    ctx->save_for_backward(std::move(save));
    ctx->saved_data["coarse"] = variant != kSparse;
    return out;
  }

  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx,
                                                 torch::autograd::variable_list grads) {
    const auto t = ctx->get_saved_variables();
    const at::Tensor dout = grads[0].contiguous();
    auto g = ::backward(t[0], t[1], t[2], t[3], dout, t[4], t[5], ctx->saved_data["coarse"].toBool(),
                        at::ArrayRef<at::Tensor>(t).slice(6));
    return {g[0], g[1], g[2], at::Tensor(), at::Tensor(), at::Tensor()};
  }
};

at::Tensor mra_attention(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, int64_t budget, int64_t variant,
                         bool prior) {
  return Attention::apply(q, k, v, budget, variant, prior);
}

template <class F>
void bind_one(const py::dict& a, const char* name, F& f) {
  f = reinterpret_cast<F>(a[name].cast<uintptr_t>());
}

void bind(const py::dict& a) {
  bind_one(a, "mra_forward_workspace_bytes", api.forward_ws);
  bind_one(a, "mra_attention_forward", api.forward);
  bind_one(a, "mra_sparse_attention_forward", api.sparse);
  bind_one(a, "mra_forward_global_workspace_bytes", api.global_ws);
  bind_one(a, "mra_attention_forward_global", api.global);
  bind_one(a, "mra_forward_pooled_rows", api.pooled_rows);
  bind_one(a, "mra_backward_workspace_bytes", api.backward_ws);
  bind_one(a, "mra_attention_backward", api.backward);
  bind_one(a, "mra_attention_backward_pooled", api.backward_pooled);
}

}  // namespace

PYBIND11_MODULE(_binding, m) {
  m.def("bind", [](const py::dict& addresses, py::object raiser) {
    bind(addresses);
    status_error = std::move(raiser);
  });
  m.def("forward", torch::wrap_pybind_function_no_gil(forward));
  m.def("mra_attention", torch::wrap_pybind_function_no_gil(mra_attention));
}
