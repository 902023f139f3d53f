// The calls of the Python binding that a program makes once per product or fit
// step, as a native module: argument checks, output allocation, the current
// stream and the C ABI call without the interpreter in between, and the
// differentiable operations (simulation, disk renderer, chi-square) as C++
// autograd functions, whose backward pass needs no Python either.  Everything
// else of the binding is Python (psflib.py, fit.py).  Per call on the host (20^2
// PSFs and scene, where the GPU waits for it): a product 8 to 11 us through ctypes,
// 3.3 to 4.8 here, of which the C call takes 3.2; a fit step through autograd 190 us,
// 110 here (77 to 120 from one process to the next, half of it torch's engine).
#include <c10/hip/HIPStream.h>
#include <torch/extension.h>

#include <string>
#include <tuple>

#include "psflib.h"

namespace {

PyObject* g_error = nullptr;   // psflib.PsflibError, kept for the life of the module
// psflib.Library and its products, kept for the life of the module
PyTypeObject* g_library = nullptr;
PyObject *g_apply = nullptr, *g_adjoint = nullptr;

// PsflibError(status, where, message), from any thread
[[noreturn]] void raise_status(psflib_status st, const char* where) {
  const std::string msg = psflib_last_error();
  py::gil_scoped_acquire gil;
  py::object exc = py::reinterpret_borrow<py::object>(g_error)((int)st, where, msg);
  PyErr_SetObject(g_error, exc.ptr());
  throw py::error_already_set();
}

void check(psflib_status st, const char* where) {
  if (st != PSFLIB_OK) raise_status(st, where);
}

[[noreturn]] void raise_value(const std::string& msg) {
  py::gil_scoped_acquire gil;
  PyErr_SetString(PyExc_ValueError, msg.c_str());
  throw py::error_already_set();
}

void* current_stream(const at::Device& d) {
  if (!d.is_cuda()) raise_value("Expected a cuda device, but got: " + d.str());
  return c10::hip::getCurrentHIPStream(d.index()).stream();
}

// a stream object (its cuda_stream), an integer, or None: the current stream
void* stream_of(py::handle stream, const at::Device& d) {
  if (stream.is_none()) return current_stream(d);
  if (py::hasattr(stream, "cuda_stream"))
    return reinterpret_cast<void*>(stream.attr("cuda_stream").cast<uintptr_t>());
  return reinterpret_cast<void*>(py::int_(py::reinterpret_borrow<py::object>(stream)).cast<uintptr_t>());
}

// What a call needs of a psflib.Library, read when it is made: a library closed
// in between gives a NULL handle, which the C ABI refuses.
struct Lib {
  const psflib_handle* h;
  int64_t ncols, M;
  at::Device device;
};

// attribute names, made once (a string for every lookup is a third of its time)
struct Names {
  PyObject *handle = PyUnicode_InternFromString("_handle"), *h = PyUnicode_InternFromString("h"),
           *ncols = PyUnicode_InternFromString("ncols"), *M = PyUnicode_InternFromString("M"),
           *device = PyUnicode_InternFromString("device"), *apply = PyUnicode_InternFromString("apply"),
           *adjoint = PyUnicode_InternFromString("apply_adjoint");
};
const Names& names() {
  static const Names* n = new Names();
  return *n;
}

py::object attr(py::handle o, PyObject* name) {
  PyObject* r = PyObject_GetAttr(o.ptr(), name);
  if (!r) throw py::error_already_set();
  return py::reinterpret_steal<py::object>(r);
}

const psflib_handle* handle_of(py::handle o) {  // o.h; with the GIL
  py::object h = attr(o, names().h);
  return h.is_none() ? nullptr : reinterpret_cast<const psflib_handle*>(h.cast<uintptr_t>());
}

// Whether o's products are those of psflib.Library: not overridden, and not replaced
// on the class or the object (a counter, a wrapper), which are called.  With the GIL.
// A fit step asks twice (in Python that took 2 us of its 130).
bool is_native(py::handle o) {
  if (!g_library || Py_TYPE(o.ptr()) != g_library ||
      PyDict_GetItem(g_library->tp_dict, names().apply) != g_apply ||
      PyDict_GetItem(g_library->tp_dict, names().adjoint) != g_adjoint)
    return false;
  py::object own = py::reinterpret_steal<py::object>(PyObject_GenericGetDict(o.ptr(), nullptr));
  if (!own) throw py::error_already_set();
  return !PyDict_GetItem(own.ptr(), names().apply) && !PyDict_GetItem(own.ptr(), names().adjoint);
}

Lib lib_of(py::handle o) {  // with the GIL
  return Lib{handle_of(o), attr(o, names().ncols).cast<int64_t>(), attr(o, names().M).cast<int64_t>(),
             attr(o, names().device).cast<at::Device>()};
}

bool is_float_on(const at::Tensor& t, const at::Device& d) {
  return t.scalar_type() == at::kFloat && t.device() == d;
}

[[noreturn]] void bad_vec(const char* name, const at::Device& d, int64_t size) {
  raise_value(std::string(name) + " must be a float32 tensor on " + d.str() + " with " +
              std::to_string(size) + " elements");
}

// x as a tensor.  What is not one has, with few exceptions, no method of this name:
// the AttributeError of a call of it.
const at::Tensor& tensor_with(py::handle x, const char* method) {
  if (!THPVariable_Check(x.ptr())) {
    (void)py::getattr(x, method);
    raise_value("a tensor is expected");
  }
  return THPVariable_Unpack(x.ptr());
}

at::Tensor vec(py::handle x, int64_t size, const at::Device& d, const char* name) {
  if (!THPVariable_Check(x.ptr())) bad_vec(name, d, size);
  const at::Tensor& t = THPVariable_Unpack(x.ptr());
  if (!is_float_on(t, d) || t.numel() != size) bad_vec(name, d, size);
  return t.contiguous();
}

// a new output tensor, or the caller's after checking that the kernels can
// write all of it and nothing past it
at::Tensor output(py::handle out, at::IntArrayRef shape, const at::Device& d) {
  if (out.is_none()) return at::empty(shape, at::TensorOptions().dtype(at::kFloat).device(d));
  int64_t numel = 1;
  for (int64_t s : shape) numel *= s;
  if (THPVariable_Check(out.ptr())) {
    const at::Tensor& t = THPVariable_Unpack(out.ptr());
    if (is_float_on(t, d) && t.is_contiguous() && t.numel() == numel) return t;
  }
  raise_value("out must be a contiguous float32 tensor on " + d.str() + " with " + std::to_string(numel) +
              " elements");
}

py::object returned(py::handle out, const at::Tensor& t) {
  return out.is_none() ? py::cast(t) : py::reinterpret_borrow<py::object>(out);
}

py::object apply(py::handle self, py::handle scene, py::handle out, py::handle stream) {
  const Lib lib = lib_of(self);
  const at::Tensor Z = vec(scene, lib.ncols, lib.device, "scene");
  const at::Tensor o = output(out, {lib.M}, lib.device);
  void* s = stream_of(stream, lib.device);
  psflib_status st;
  {
    py::gil_scoped_release nogil;
    st = psflib_apply(lib.h, Z.data_ptr<float>(), o.data_ptr<float>(), s);
  }
  check(st, "psflib_apply");
  return returned(out, o);
}

py::object apply_adjoint(py::handle self, py::handle g, py::handle out, py::handle stream) {
  const Lib lib = lib_of(self);
  const at::Tensor G = vec(g, lib.M, lib.device, "g");
  const at::Tensor o = output(out, {lib.ncols}, lib.device);
  void* s = stream_of(stream, lib.device);
  psflib_status st;
  {
    py::gil_scoped_release nogil;
    st = psflib_apply_adjoint(lib.h, G.data_ptr<float>(), o.data_ptr<float>(), s);
  }
  check(st, "psflib_apply_adjoint");
  return returned(out, o);
}

py::object apply_batched(py::handle self, py::handle scenes, py::handle out, py::handle stream) {
  const Lib lib = lib_of(self);
  const bool tensor = THPVariable_Check(scenes.ptr());
  at::Tensor Z;
  if (tensor) Z = THPVariable_Unpack(scenes.ptr());
  if (!tensor || !is_float_on(Z, lib.device) || Z.dim() != 2 || Z.size(1) != lib.ncols)
    raise_value("scenes must be a float32 tensor [B][" + std::to_string(lib.ncols) + "] on " +
                lib.device.str());
  Z = Z.contiguous();
  const int64_t B = Z.size(0);
  const at::Tensor o = output(out, {B, lib.M}, lib.device);
  void* s = stream_of(stream, lib.device);
  psflib_status st;
  {
    py::gil_scoped_release nogil;
    st = psflib_apply_batched(lib.h, Z.data_ptr<float>(), o.data_ptr<float>(), (int32_t)B, s);
  }
  check(st, "psflib_apply_batched");
  return returned(out, o);
}

// ------------------------------------------------------------- autograd ----
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// What a graph holds of a library: its handle object (psflib._Handle), whose handle is
// read when it is used, and the library itself weakly.  Released with the GIL.
struct LibRef : torch::CustomClassHolder {
  py::object handle, library;
  Lib lib;  // when the forward pass ran
  explicit LibRef(py::handle o)
      : handle(attr(o, names().handle)), library(py::weakref(o)), lib(lib_of(o)) {}
  ~LibRef() override {
    if (!Py_IsInitialized()) {
      handle.release();
      library.release();
      return;
    }
    py::gil_scoped_acquire gil;
    handle = py::object();
    library = py::object();
  }
};

at::Tensor product(const Lib& lib, bool adjoint, const at::Tensor& x, const char* name) {
  const int64_t in = adjoint ? lib.M : lib.ncols;
  if (!is_float_on(x, lib.device) || x.numel() != in) bad_vec(name, lib.device, in);
  const at::Tensor o = at::empty({adjoint ? lib.ncols : lib.M}, x.options().memory_format(std::nullopt));
  void* s = current_stream(lib.device);
  if (adjoint)
    check(psflib_apply_adjoint(lib.h, x.data_ptr<float>(), o.data_ptr<float>(), s), "psflib_apply_adjoint");
  else
    check(psflib_apply(lib.h, x.data_ptr<float>(), o.data_ptr<float>(), s), "psflib_apply");
  return o;
}

struct Simulate : torch::autograd::Function<Simulate> {
  static at::Tensor forward(AutogradContext* ctx, const at::Tensor& Z, c10::intrusive_ptr<LibRef> ref) {
    ctx->saved_data["lib"] = c10::IValue::make_capsule(ref);
    return product(ref->lib, false, Z.contiguous(), "scene");
  }
  static variable_list backward(AutogradContext* ctx, variable_list g) {
    auto ref = c10::static_intrusive_pointer_cast<LibRef>(ctx->saved_data["lib"].toCapsule());
    const at::Tensor gS = g[0].contiguous().to(at::kFloat);
    Lib lib = ref->lib;
    {
      py::gil_scoped_acquire gil;
      const py::object o = ref->library();
      if (!o.is_none() && !is_native(o))
        // another adjoint than the class's has been put in its place
        return {o.attr("apply_adjoint")(gS).cast<at::Tensor>(), at::Tensor()};
      lib.h = handle_of(ref->handle);
    }
    return {product(lib, true, gS, "g"), at::Tensor()};
  }
};

at::Tensor simulate(py::handle lib, py::handle scene) {
  const at::Tensor Z = tensor_with(scene, "contiguous");
  auto ref = c10::make_intrusive<LibRef>(lib);
  py::gil_scoped_release nogil;
  return Simulate::apply(Z, std::move(ref));
}

at::Tensor render(const at::Tensor& th, int64_t N, double S, double rmax) {
  at::Tensor Z = at::empty({N * N}, th.options().dtype(at::kFloat));
  check(psflib_render_disk((int32_t)N, S, rmax, th.data_ptr<double>(), Z.data_ptr<float>(),
                           current_stream(th.device())),
        "psflib_render_disk");
  return Z;
}

at::Tensor render_grad(const at::Tensor& th, int64_t N, double S, double rmax, const at::Tensor& dZ) {
  at::Tensor dth = at::empty({5}, th.options());
  check(psflib_render_disk_grad((int32_t)N, S, rmax, th.data_ptr<double>(), dZ.data_ptr<float>(),
                                dth.data_ptr<double>(), current_stream(th.device())),
        "psflib_render_disk_grad");
  return dth;
}

struct RenderDisk : torch::autograd::Function<RenderDisk> {
  static at::Tensor forward(AutogradContext* ctx, const at::Tensor& theta, int64_t N, double S, double rmax) {
    const at::Tensor th = theta.detach().to(at::kDouble).contiguous();
    ctx->save_for_backward({th});
    ctx->saved_data["N"] = N;
    ctx->saved_data["S"] = S;
    ctx->saved_data["rmax"] = rmax;
    return render(th, N, S, rmax);
  }
  static variable_list backward(AutogradContext* ctx, variable_list g) {
    const at::Tensor th = ctx->get_saved_variables()[0];
    const at::Tensor dZ = g[0].contiguous().to(at::kFloat);
    return {render_grad(th, ctx->saved_data["N"].toInt(), ctx->saved_data["S"].toDouble(),
                        ctx->saved_data["rmax"].toDouble(), dZ),
            at::Tensor(), at::Tensor(), at::Tensor()};
  }
};

// the disk's parameters: the kernels read five values
const at::Tensor& disk_parameters(py::handle theta) {
  const at::Tensor& t = tensor_with(theta, "detach");
  if (t.numel() < 5) raise_value("theta must have 5 elements, got " + std::to_string(t.numel()));
  return t;
}

at::Tensor render_disk(py::handle theta, int64_t N, double S, double rmax) {
  const at::Tensor th = disk_parameters(theta);
  py::gil_scoped_release nogil;
  return RenderDisk::apply(th, N, S, rmax);
}

at::Tensor float64_vec(py::handle x, const char* name, int64_t M, const at::Device& d) {
  if (THPVariable_Check(x.ptr())) {
    const at::Tensor& t = THPVariable_Unpack(x.ptr());
    if (t.scalar_type() == at::kDouble && t.device() == d && t.numel() == M) return t.contiguous();
  }
  raise_value(std::string(name) + " must be a float64 tensor of " + std::to_string(M) + " elements on " +
              d.str());
}

// (loss, dL/dS)
std::tuple<at::Tensor, at::Tensor> misfit(const at::Tensor& S, const at::Tensor& D, const at::Tensor& V,
                                          double K) {
  const int64_t M = S.numel();
  at::Tensor loss = at::empty({}, D.options().memory_format(std::nullopt));
  at::Tensor grad = at::empty_like(S);
  check(psflib_chi2(M, K, S.data_ptr<float>(), D.data_ptr<double>(), V.data_ptr<double>(),
                    loss.data_ptr<double>(), grad.data_ptr<float>(), current_stream(S.device())),
        "psflib_chi2");
  return {loss, grad};
}

struct Chi2 : torch::autograd::Function<Chi2> {
  static at::Tensor forward(AutogradContext* ctx, const at::Tensor& model, const at::Tensor& D,
                            const at::Tensor& V, double K) {
    auto [loss, grad] = misfit(model.detach().contiguous(), D, V, K);
    ctx->save_for_backward({grad});
    return loss;
  }
  static variable_list backward(AutogradContext* ctx, variable_list gL) {
    const at::Tensor grad = ctx->get_saved_variables()[0];
    return {grad * gL[0].to(grad.scalar_type()), at::Tensor(), at::Tensor(), at::Tensor()};
  }
};

at::Tensor chi2(py::handle model, py::handle counts, py::handle var, double K) {
  const at::Tensor S = tensor_with(model, "detach");
  if (S.scalar_type() != at::kFloat) raise_value("model must be a float32 image");
  const at::Tensor D = float64_vec(counts, "counts", S.numel(), S.device());
  const at::Tensor V = float64_vec(var, "var", S.numel(), S.device());
  py::gil_scoped_release nogil;
  return Chi2::apply(S, D, V, K);
}

std::tuple<at::Tensor, at::Tensor> loss_and_grad(py::handle self, py::handle theta, py::handle counts,
                                                 py::handle var, double K, double rmax) {
  const Lib lib = lib_of(self);
  const int64_t N = self.attr("N").cast<int64_t>();
  const double S = self.attr("S").cast<double>();
  at::Tensor th = disk_parameters(theta);
  const at::Tensor D = float64_vec(counts, "counts", lib.M, lib.device);
  const at::Tensor V = float64_vec(var, "var", lib.M, lib.device);
  py::gil_scoped_release nogil;
  th = th.detach().to(D.device(), at::kDouble).contiguous();
  const at::Tensor image = product(lib, false, render(th, N, S, rmax), "scene");
  auto [loss, gS] = misfit(image, D, V, K);
  const at::Tensor gZ = product(lib, true, gS, "g");
  return {loss, render_grad(th, N, S, rmax, gZ)};
}

}  // namespace

PYBIND11_MODULE(_psfop, m) {
  m.doc() = "Native calls of the psflib binding.";
  m.def("set_error", [](py::object cls) { g_error = cls.release().ptr(); });
  m.def("set_library", [](py::object cls) {
    g_apply = py::object(cls.attr("apply")).release().ptr();
    g_adjoint = py::object(cls.attr("apply_adjoint")).release().ptr();
    g_library = reinterpret_cast<PyTypeObject*>(cls.release().ptr());
  });
  m.def("is_native", &is_native);
  m.def("current_stream", [](const at::Device& d) { return reinterpret_cast<uintptr_t>(current_stream(d)); });
  m.def("apply", &apply);
  m.def("apply_adjoint", &apply_adjoint);
  m.def("apply_batched", &apply_batched);
  m.def("simulate", &simulate);
  m.def("render_disk", &render_disk);
  m.def("chi2", &chi2);
  m.def("loss_and_grad", &loss_and_grad);
}
