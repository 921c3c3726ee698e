// The differentiable call of the package (autograd.py) in native code: checks, output tensors and bookkeeping around
// skrull_attn_fwd and skrull_attn_bwd.  A pass of 932 tokens, 4/4 heads of 64, forward and gradients, takes the GPU 34 us;
// written in Python the calls around it kept the host busy for 50 us in a process whose threads run close to each other and
// 107 in one where they do not (the backward runs in a thread of the autograd engine, and every Python object it touches
// moves between the two).  36 and 70 this way; torch's own a + b and its gradient take 30 and 42.

#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <memory>

#include "skrull_attn.h"

namespace {

using torch::autograd::AutogradContext;
using torch::autograd::Variable;
using torch::autograd::variable_list;

PyObject *g_check = nullptr;  // binding._check: raises what an error code stands for

// A binding.Plan, kept by the graph.  Its handle is read when it is needed: the program may destroy the plan before.
struct PlanObject {
    PyObject *plan;
    explicit PlanObject(PyObject *p) : plan(p) { Py_INCREF(p); }
    ~PlanObject()
    {
        if (!Py_IsInitialized()) return;
        const PyGILState_STATE gil = PyGILState_Ensure();
        Py_DECREF(plan);
        PyGILState_Release(gil);
    }
    PlanObject(const PlanObject &) = delete;
    PlanObject &operator=(const PlanObject &) = delete;
};

// The handle of a plan, null for one that is destroyed.  With the GIL held.
const skrull_attn_plan_t *handle_of(PyObject *plan)
{
    PyObject *handle = PyObject_GetAttrString(plan, "handle");
    if (!handle) throw python_error();
    void *p = nullptr;
    if (handle != Py_None) {
        PyObject *value = PyObject_GetAttrString(handle, "value");  // (a ctypes.c_void_p)
        if (value && value != Py_None) p = PyLong_AsVoidPtr(value);
        Py_XDECREF(value);
    }
    Py_DECREF(handle);
    if (PyErr_Occurred()) throw python_error();
    return (const skrull_attn_plan_t *)p;
}

void check(int rc)
{
    if (rc == SKRULL_OK) return;
    const PyGILState_STATE gil = PyGILState_Ensure();
    PyObject *r = PyObject_CallFunction(g_check, "i", rc);
    Py_XDECREF(r);
    python_error error;
    error.persist();
    PyGILState_Release(gil);
    throw error;
}

void *current_stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

struct Attention : torch::autograd::Function<Attention> {
    static Variable forward(AutogradContext *ctx, const Variable &q, const Variable &k, const Variable &v, const std::shared_ptr<PlanObject> &plan,
                            const skrull_attn_plan_t *handle, int64_t q_heads, int64_t total_q)
    {
        at::Tensor o = at::empty_like(q), lse = at::empty({q_heads, total_q}, q.options().dtype(at::kFloat));
        check(skrull_attn_fwd(handle, q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (float *)lse.data_ptr(), current_stream()));
        ctx->saved_data["plan"] = c10::IValue::make_capsule(c10::make_intrusive<Holder>(plan));
        ctx->save_for_backward({q, k, v, o, lse});
        return o;
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        const variable_list saved = ctx->get_saved_variables();
        const at::Tensor &q = saved[0], &k = saved[1], &v = saved[2], &o = saved[3], &lse = saved[4];
        const auto holder = c10::static_intrusive_pointer_cast<Holder>(ctx->saved_data["plan"].toCapsule());
        const skrull_attn_plan_t *handle;
        {
            const PyGILState_STATE gil = PyGILState_Ensure();
            try {
                handle = handle_of(holder->plan->plan);
            } catch (python_error &e) {
                e.persist();
                PyGILState_Release(gil);
                throw;
            }
            PyGILState_Release(gil);
        }
        skrull_attn_plan_info_t info;
        check(skrull_attn_plan_info(handle, &info));
        const at::Tensor d_o = grads[0].contiguous();
        at::Tensor dq = at::empty_like(q), dk = at::empty_like(k), dv = at::empty_like(v);
        const int64_t bytes = std::max<int64_t>(info.bwd_workspace_bytes, 16);
        at::Tensor ws = at::empty({bytes}, q.options().dtype(at::kByte));
        check(skrull_attn_bwd(handle, q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (const float *)lse.data_ptr(), d_o.data_ptr(),
                              dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), ws.data_ptr(), (size_t)bytes, current_stream()));
        return {dq, dk, dv, at::Tensor(), at::Tensor(), at::Tensor(), at::Tensor()};
    }
    struct Holder : torch::CustomClassHolder {
        std::shared_ptr<PlanObject> plan;
        explicit Holder(std::shared_ptr<PlanObject> p) : plan(std::move(p)) {}
    };
};

// attention(q, k, v, plan, total_q, total_k, q_heads, kv_heads, head_dim)
PyObject *attention(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 9 || !THPVariable_Check(args[0]) || !THPVariable_Check(args[1]) || !THPVariable_Check(args[2])) {
        PyErr_SetString(PyExc_TypeError, "attention(q, k, v, plan, total_q, total_k, q_heads, kv_heads, head_dim)");
        return nullptr;
    }
    const at::Tensor &q = THPVariable_Unpack(args[0]), &k = THPVariable_Unpack(args[1]), &v = THPVariable_Unpack(args[2]);
    int64_t size[5];
    for (int i = 0; i < 5; ++i) size[i] = PyLong_AsLongLong(args[4 + i]);
    if (PyErr_Occurred()) return nullptr;
    for (const at::Tensor *t : {&q, &k, &v})
        if (!t->is_cuda() || t->scalar_type() != at::kBFloat16 || !t->is_contiguous()) {
            PyErr_SetString(PyExc_ValueError, "q, k, v must be contiguous bf16 CUDA tensors");
            return nullptr;
        }
    const int64_t q_shape[3] = {size[0], size[2], size[4]}, k_shape[3] = {size[1], size[3], size[4]};
    if (q.sizes() != at::IntArrayRef(q_shape, 3) || k.sizes() != at::IntArrayRef(k_shape, 3) || v.sizes() != k.sizes()) {
        PyErr_SetString(PyExc_ValueError, "tensor shapes do not match the plan");
        return nullptr;
    }
    const skrull_attn_plan_t *handle = handle_of(args[3]);
    auto plan = std::make_shared<PlanObject>(args[3]);
    at::Tensor o;
    {
        pybind11::gil_scoped_release no_gil;
        o = Attention::apply(q, k, v, plan, handle, size[2], size[0]);
    }
    return THPVariable_Wrap(std::move(o));
    END_HANDLE_TH_ERRORS
}

PyObject *set_check(PyObject *, PyObject *f)
{
    Py_INCREF(f);
    Py_XSETREF(g_check, f);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"attention", (PyCFunction)(void (*)())attention, METH_FASTCALL, "the differentiable call"},
                         {"set_check", set_check, METH_O, "the callable that raises what an error code stands for"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_autograd", "autograd of skrull_attn", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__autograd() { return PyModule_Create(&module); }
