// Argument marshalling of the calls a manager makes every period, for binding.py: tensors to device pointers, the current
// stream, the C call.  What a call costs the host is all that three of them (anticipator, look-ahead map, scaler over 4096
// requests) take, 10 us each through ctypes: four attributes of every tensor, seventeen converted arguments, a stream object.
// Host time of the calls of a management period, ctypes / so: 29.5 / 10.0 us; the period itself 31.8 -> 23.8 us, which is what
// its three launches take on the GPU.
//
// Only calls with nothing to object to are made here: tensors of the plain type, on the GPU, contiguous, of the right type and
// size, integers that fit.  Anything else returns NotImplemented with nothing done, and binding.py goes its own way, which
// says what is wrong.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "preserve.h"

namespace {

PyObject *g_raw_stream, *g_device;   // torch._C._cuda_getCurrentRawStream, _cuda_getDevice

// The library's calls, by the addresses that binding.py has from the library it loaded.
struct Calls {
    decltype(&ps_predict_load) predict_load;
    decltype(&ps_anticipate) anticipate;
    decltype(&ps_anticipate_static) anticipate_static;
    decltype(&ps_lookahead_update) lookahead_update;
    decltype(&ps_scaler_scan) scaler_scan;
    decltype(&ps_route) route;
    decltype(&ps_forecast) forecast;
} g_calls;

PyObject* bind(PyObject*, PyObject* const* at, Py_ssize_t n) {
    void* p[7];
    if (n != 7) { PyErr_SetString(PyExc_TypeError, "bind: seven addresses"); return nullptr; }
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(at[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    g_calls = {(decltype(&ps_predict_load))p[0], (decltype(&ps_anticipate))p[1], (decltype(&ps_anticipate_static))p[2],
               (decltype(&ps_lookahead_update))p[3], (decltype(&ps_scaler_scan))p[4], (decltype(&ps_route))p[5],
               (decltype(&ps_forecast))p[6]};
    Py_RETURN_NONE;
}

struct Args {
    PyObject* const* at;
    bool good = true;

    // A tensor's device pointer (null for None); n: its elements, if not null.
    template <typename T>
    T* tensor(int i, at::ScalarType type, int64_t* n = nullptr, bool optional = false) {
        if (n) *n = -1;
        PyObject* o = at[i];
        if (o == Py_None && optional) return nullptr;
        if (!good || !THPVariable_CheckExact(o)) { good = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) { good = false; return nullptr; }
        if (n) *n = t.numel();
        return (T*)t.data_ptr();
    }
    template <typename T>
    T* sized(int i, at::ScalarType type, int64_t want, bool optional = false) {
        int64_t n;
        T* p = tensor<T>(i, type, &n, optional);
        if (n >= 0 && n != want) good = false;
        return p;
    }
    int32_t i32(int i) {
        if (!good || !PyLong_CheckExact(at[i])) { good = false; return 0; }
        int overflow = 0;
        const long v = PyLong_AsLongAndOverflow(at[i], &overflow);
        if (overflow || v != (int32_t)v) { good = false; return 0; }
        return (int32_t)v;
    }
    // a count of elements that the call takes as an int32
    int32_t count32(int64_t n) {
        if (n != (int32_t)n) good = false;
        return (int32_t)n;
    }
    void* pointer(int i) {
        if (!good || !PyLong_CheckExact(at[i])) { good = false; return nullptr; }
        void* p = PyLong_AsVoidPtr(at[i]);
        if (PyErr_Occurred()) { PyErr_Clear(); good = false; }
        return p;
    }
};

constexpr at::ScalarType kI32 = at::kInt, kI64 = at::kLong, kF32 = at::kFloat, kF64 = at::kDouble, kU8 = at::kByte;

// The current stream of the current device; false with an exception set if torch cannot say.
bool current_stream(void** s) {
    PyObject* dev = PyObject_CallNoArgs(g_device);
    if (!dev) return false;
    PyObject* raw = PyObject_CallOneArg(g_raw_stream, dev);
    Py_DECREF(dev);
    if (!raw) return false;
    *s = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    return !PyErr_Occurred();
}

// parse: fills in the arguments and returns the call (given the stream), which is made without the interpreter's lock.
template <typename Parse>
PyObject* make_call(PyObject* const* at, Py_ssize_t n, Py_ssize_t want, Parse parse) {
    if (n != want) Py_RETURN_NOTIMPLEMENTED;
    try {
        Args a{at};
        auto call = parse(a);
        if (!a.good) Py_RETURN_NOTIMPLEMENTED;
        void* stream;
        if (!current_stream(&stream)) return nullptr;
        int code = PS_OK;
        bool thrown = false;
        Py_BEGIN_ALLOW_THREADS
        try {
            code = call(stream);
        } catch (...) {                      // (out of memory: the lock has to be taken again all the same)
            thrown = true;
        }
        Py_END_ALLOW_THREADS
        if (thrown) return PyErr_NoMemory();
        return PyLong_FromLong(code);
    } catch (...) {                          // a tensor without storage, say
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    }
}

PyObject* predict_load(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 8, [](Args& a) {
        int64_t tokens = 0, offs = 0, ws = 0;
        const ps_model* model = (const ps_model*)a.pointer(0);
        const int32_t* ids = a.tensor<int32_t>(1, kI32, &tokens);
        const int32_t* offsets = a.tensor<int32_t>(2, kI32, &offs);
        const int32_t* lengths = a.tensor<int32_t>(3, kI32, nullptr, true);
        float* pred_f = a.tensor<float>(4, kF32);
        int32_t* pred_tokens = a.tensor<int32_t>(5, kI32);
        void* workspace = a.tensor<void>(6, kU8, &ws);
        ps_status* st = a.tensor<ps_status>(7, kI64, nullptr, true);
        const int32_t n_req = a.count32(offs - 1);
        return [=](void* s) {
            return g_calls.predict_load((ps_model*)model, ids, offsets, lengths, n_req, tokens, pred_f, pred_tokens, workspace, (size_t)ws, st, s);
        };
    });
}

PyObject* anticipate(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 10, [](Args& a) {
        int64_t req = 0, ws = 0;
        const int32_t* pred = a.tensor<int32_t>(0, kI32, &req);
        const int32_t* inst = a.sized<int32_t>(1, kI32, req);
        const int32_t* arrival = a.sized<int32_t>(2, kI32, req);
        const int32_t n_inst = a.i32(4), horizon = a.i32(5);
        const int32_t* rate = a.sized<int32_t>(3, kI32, n_inst, true);
        int32_t* load = a.sized<int32_t>(6, kI32, (int64_t)n_inst * horizon);
        int64_t* overflow = a.sized<int64_t>(7, kI64, n_inst, true);
        void* workspace = a.tensor<void>(8, kU8, &ws);
        ps_status* st = a.tensor<ps_status>(9, kI64, nullptr, true);
        return [=](void* s) {
            return g_calls.anticipate(pred, inst, arrival, rate, req, n_inst, horizon, load, overflow, workspace, (size_t)ws, st, s);
        };
    });
}

PyObject* anticipate_static(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 9, [](Args& a) {
        int64_t req = 0;
        const int32_t* pred = a.tensor<int32_t>(0, kI32, &req);
        const int32_t* inst = a.sized<int32_t>(1, kI32, req);
        const int32_t* arrival = a.sized<int32_t>(2, kI32, req);
        const int32_t n_inst = a.i32(4), horizon = a.i32(5);
        const int32_t* rate = a.sized<int32_t>(3, kI32, n_inst, true);
        int32_t* load = a.sized<int32_t>(6, kI32, (int64_t)n_inst * horizon);
        int64_t* overflow = a.sized<int64_t>(7, kI64, n_inst, true);
        ps_status* st = a.tensor<ps_status>(8, kI64, nullptr, true);
        return [=](void* s) { return g_calls.anticipate_static(pred, inst, arrival, rate, req, n_inst, horizon, load, overflow, st, s); };
    });
}

PyObject* lookahead_update(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 14, [](Args& a) {
        int64_t rec = 0, ws = 0;
        const int32_t* cols[6];
        cols[0] = a.tensor<int32_t>(0, kI32, &rec);
        for (int i = 1; i < 6; ++i) cols[i] = a.sized<int32_t>(i, kI32, rec);
        const int32_t n_inst = a.i32(6), map_len = a.i32(7);
        int32_t* kv = a.sized<int32_t>(8, kI32, (int64_t)n_inst * map_len);
        int64_t* overflow = a.sized<int64_t>(9, kI64, n_inst, true);
        void* workspace = a.tensor<void>(10, kU8, &ws);
        const int32_t* capacity = a.sized<int32_t>(11, kI32, n_inst, true);
        float* fraction = a.sized<float>(12, kF32, (int64_t)n_inst * map_len, true);
        ps_status* st = a.tensor<ps_status>(13, kI64, nullptr, true);
        const int32_t *c0 = cols[0], *c1 = cols[1], *c2 = cols[2], *c3 = cols[3], *c4 = cols[4], *c5 = cols[5];
        return [=](void* s) {
            return g_calls.lookahead_update(c0, c1, c2, c3, c4, c5, rec, n_inst, map_len, kv, overflow, capacity, fraction, workspace,
                                       (size_t)ws, st, s);
        };
    });
}

PyObject* scaler_scan(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 13, [](Args& a) {
        const int32_t n_inst = a.i32(2), map_len = a.i32(3), window = a.i32(4);
        const int32_t* kv = a.sized<int32_t>(0, kI32, (int64_t)n_inst * map_len);
        const int32_t* capacity = a.sized<int32_t>(1, kI32, n_inst);
        int32_t* over_count = a.sized<int32_t>(5, kI32, n_inst);
        int32_t* peak = a.sized<int32_t>(6, kI32, n_inst);
        int32_t* overloaded = a.sized<int32_t>(7, kI32, n_inst);
        int32_t* summary = a.sized<int32_t>(8, kI32, 2);
        double* scale_down = a.sized<double>(9, kF64, 1);
        const int32_t over_pct = a.i32(10), share_pct = a.i32(11), idle_pct = a.i32(12);
        return [=](void* s) {
            return g_calls.scaler_scan(kv, capacity, n_inst, map_len, window, over_pct, share_pct, idle_pct, over_count, peak, overloaded,
                                  summary, scale_down, s);
        };
    });
}

PyObject* route(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 13, [](Args& a) {
        int64_t req = 0;
        const int32_t* prompt = a.tensor<int32_t>(0, kI32, &req);
        const int32_t* pred = a.sized<int32_t>(1, kI32, req);
        const int32_t n_inst = a.i32(2), window = a.i32(3);
        int32_t* windows = a.sized<int32_t>(4, kI32, (int64_t)n_inst * window, true);
        const int32_t* capacity = a.sized<int32_t>(5, kI32, n_inst);
        int64_t* queued = a.sized<int64_t>(6, kI64, n_inst);
        int64_t* current = a.sized<int64_t>(7, kI64, n_inst);
        int32_t* assigned = a.sized<int32_t>(8, kI32, req);
        int64_t* score = a.sized<int64_t>(9, kI64, req);
        const int32_t t_mem = a.i32(10), beta = a.i32(11);
        ps_status* st = a.tensor<ps_status>(12, kI64, nullptr, true);
        const int32_t n_req = a.count32(req);
        return [=](void* s) {
            return g_calls.route(prompt, pred, n_req, n_inst, window, windows, capacity, queued, current, t_mem, beta, assigned, score, st, s);
        };
    });
}

PyObject* forecast(PyObject*, PyObject* const* at, Py_ssize_t n) {
    return make_call(at, n, 8, [](Args& a) {
        const int32_t hidden = a.i32(1), services = a.i32(4), k = a.i32(5);
        const int64_t h = hidden, model = 5 * h * h + 10 * h + 1;
        if (h < 0 || h > 4096) a.good = false;
        const float* weights = a.sized<float>(0, kF32, services * 2ll * model);
        const float* hist_p = a.sized<float>(2, kF32, (int64_t)services * k);
        const float* hist_d = a.sized<float>(3, kF32, (int64_t)services * k);
        const float* mu = a.sized<float>(6, kF32, 3ll * services);
        float* out = a.sized<float>(7, kF32, 5ll * services);
        return [=](void* s) { return g_calls.forecast(weights, hidden, hist_p, hist_d, services, k, mu, out, s); };
    });
}

#define PS_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PS_METHOD(bind), PS_METHOD(predict_load), PS_METHOD(anticipate), PS_METHOD(anticipate_static), PS_METHOD(lookahead_update),
                         PS_METHOD(scaler_scan), PS_METHOD(route), PS_METHOD(forecast), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject* torch_c = PyImport_ImportModule("torch._C");
    if (!torch_c) return nullptr;
    g_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
    g_device = g_raw_stream ? PyObject_GetAttrString(torch_c, "_cuda_getDevice") : nullptr;
    Py_DECREF(torch_c);
    if (!g_device) return nullptr;
    return PyModule_Create(&module);
}
