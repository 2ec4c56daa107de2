// The argument marshalling of binding.py's calls in native code: checks, fresh outputs and the C call of one entry point per
// function, for the ordinary form of a call.  What is not of that form -- another tensor type or place, a shape or an output
// that does not fit, numbers that are not Python numbers -- is declined (None) before anything has happened, and binding.py
// goes through it step by step, with its own checks and messages.  A call that the library refuses returns its code.
// Everything that can fail, the Python objects of the results included, is done before the library is called: a failure behind
// the launch, taken for a declined call, would have binding.py launch it a second time.
//
// Why: of the 26 us of the smallest stage-1 call 18 were Python (eleven outputs and a workspace of 1.2 us each, 31 ctypes
// arguments), of one pruning level's 28 us of host time 15; the kernels of both take less than that.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <vector>

#include "metok.h"

namespace {

// Thrown and caught inside this file only.  A Python error is never a reason to decline: it may be a signal's exception.
struct Declined {};
struct Raised {};                          // a Python error is set

// ---- reading arguments -----------------------------------------------------------------------------------------------
inline void need(bool ok) { if (!ok) throw Declined(); }

inline int64_t integer(PyObject* o) {
    need(PyLong_CheckExact(o) || PyBool_Check(o));
    int overflow = 0;
    const int64_t v = PyLong_AsLongLongAndOverflow(o, &overflow);
    need(!overflow);
    return v;
}
inline int int32(PyObject* o) {
    const int64_t v = integer(o);
    need(v >= INT32_MIN && v <= INT32_MAX);
    return static_cast<int>(v);
}
inline double real(PyObject* o) {
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    return static_cast<double>(int32(o));
}
inline bool given(PyObject* o) { return o != Py_None; }

struct Owned {                             // a reference of our own, to what a Python function returned
    PyObject* o;
    explicit Owned(PyObject* p) : o(p) { if (!o) throw Raised(); }
    Owned(const Owned&) = delete;
    ~Owned() { Py_XDECREF(o); }
    PyObject* release() { PyObject* p = o; o = nullptr; return p; }
};

// A plain tensor on the GPU, contiguous.
inline const at::Tensor& tensor(PyObject* o) {
    need(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    need(t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous());
    return t;
}
inline void* address(const at::Tensor& t) { return t.data_ptr(); }
inline int dtype_code(const at::Tensor& t) {
    const auto s = t.scalar_type();
    need(s == at::kBFloat16 || s == at::kFloat);
    return s == at::kBFloat16 ? METOK_BF16 : METOK_F32;
}

// The caller's outputs: None, or a dict.
struct Outputs {
    PyObject* dict;                        // borrowed, nullptr: none given
    at::Device device;
    Outputs(PyObject* o, const at::Tensor& like) : dict(given(o) ? o : nullptr), device(like.device()) { need(!dict || PyDict_CheckExact(dict)); }
    PyObject* find(const char* name) const {
        if (!dict) return nullptr;
        const Owned key(PyUnicode_FromString(name));
        PyObject* v = PyDict_GetItemWithError(dict, key.o);  // borrowed
        if (!v && PyErr_Occurred()) throw Raised();
        return v && given(v) ? v : nullptr;
    }
    at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type) const {
        for (const int64_t n : shape) need(n >= 0);
        return at::empty(shape, at::TensorOptions().dtype(type).device(device));
    }
    at::Tensor get(const char* name, at::IntArrayRef shape, at::ScalarType type) const {
        if (PyObject* v = find(name)) {
            const at::Tensor& t = tensor(v);
            need(t.scalar_type() == type && t.sizes() == shape);
            return t;
        }
        return fresh(shape, type);
    }
};
inline at::Tensor workspace_of(PyObject* o, const Outputs& out, size_t bytes) {
    if (given(o)) return tensor(o);
    return out.fresh({static_cast<int64_t>(std::max<size_t>(bytes, 256))}, at::kByte);
}

// ---- results -----------------------------------------------------------------------------------------------------------
struct Result : Owned {
    Result() : Owned(PyDict_New()) {}
    void put(const char* name, PyObject* v) {                // takes the reference
        const Owned own(v);
        if (PyDict_SetItemString(o, name, v)) throw Raised();
    }
    void put(const char* name, const at::Tensor& t) { put(name, THPVariable_Wrap(t)); }
};

// A call with its arguments, pointers among them, read now.
template <typename F, typename... A> auto bound(F f, A... a) { return [=] { return f(a...); }; }

// The library call of one native call, without the interpreter's lock, as ctypes does.
struct Launch {
    bool made = false;
    template <typename F> int operator()(F&& call) {
        struct Released {
            PyThreadState* state = PyEval_SaveThread();
            ~Released() { PyEval_RestoreThread(state); }
        } released;
        made = true;
        return call();
    }
};
// The library's code, unless it is 0: then the results.
inline PyObject* answer(int rc, Owned& results) { return rc ? PyLong_FromLong(rc) : results.release(); }

template <typename F> PyObject* guarded(Py_ssize_t nargs, Py_ssize_t expected, F&& body) {
    if (nargs != expected) { PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", expected, nargs); return nullptr; }
    Launch launch;
    try {
        return body(launch);
    } catch (const Raised&) {
        return nullptr;
    } catch (python_error& e) {            // torch's form of the same
        e.restore();
        return nullptr;
    } catch (const Declined&) {
        Py_RETURN_NONE;
    } catch (const std::exception& e) {    // an allocation that failed, for instance: the step-by-step path reports it
        if (launch.made) { PyErr_SetString(PyExc_RuntimeError, e.what()); return nullptr; }      // not again
        Py_RETURN_NONE;
    }
}
// binding.py's function for the current stream's handle, asked once everything else fits.
inline void* stream_of(PyObject* f) {
    const Owned handle(PyObject_CallNoArgs(f));
    return reinterpret_cast<void*>(integer(handle.o));
}

// ---- stage 1 -----------------------------------------------------------------------------------------------------------
// feats, grid_h, grid_w, k, text_emb, alpha, beta, s1, s2, sim_mode, event_reduce, pool_edge, workspace, out, stream
template <bool BATCHED>
PyObject* segment_compress(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 15, [&](Launch& launch) -> PyObject* {
        const at::Tensor& feats = tensor(a[0]);
        const at::Tensor& text = tensor(a[4]);
        need(feats.dim() == (BATCHED ? 4 : 3));
        const int64_t B = BATCHED ? feats.size(0) : 1, T = feats.size(BATCHED), N = feats.size(BATCHED + 1), d = feats.size(BATCHED + 2);
        const int64_t limit = INT32_MAX;
        need(B <= limit && T <= limit && N <= limit && d <= limit);
        const int gh = int32(a[1]), gw = int32(a[2]), k = int32(a[3]), s1 = int32(a[7]), s2 = int32(a[8]);
        const double alpha = real(a[5]), beta = real(a[6]);
        const int sim_mode = int32(a[9]), reduce = int32(a[10]), edge = int32(a[11]), dt = dtype_code(feats);
        need(static_cast<int64_t>(gh) * gw == N);
        if (BATCHED) need(text.dim() == 2 && text.size(0) == B && text.size(1) == d);
        const int64_t cap = metok_compress_encoder_tokens_capacity_rows(static_cast<int>(T), gh, gw, s1, s2, edge);
        need(cap >= 0 && k >= 0);
        const Outputs out(a[13], feats);
        at::Tensor tokens;
        if (PyObject* v = out.find("out_tokens")) {
            tokens = tensor(v);
            need(tokens.dim() == (BATCHED ? 3 : 2) && tokens.size(BATCHED + 1) == d && (!BATCHED || tokens.size(0) == B));
        } else {
            tokens = BATCHED ? out.fresh({B, cap, d}, feats.scalar_type()) : out.fresh({cap, d}, feats.scalar_type());
        }
        const int odt = dtype_code(tokens);
        const int64_t rows = tokens.size(BATCHED);
        const at::Tensor ws = workspace_of(a[12], out, BATCHED ? metok_segment_compress_batched_workspace_bytes(static_cast<int>(B), static_cast<int>(T), gh, gw, static_cast<int>(d), dt)
                                                               : metok_segment_compress_workspace_bytes(static_cast<int>(T), gh, gw, static_cast<int>(d), dt));
        auto get = [&](const char* name, int64_t len, at::ScalarType type) {
            const int64_t shape[2] = {B, len};
            return out.get(name, BATCHED ? at::IntArrayRef(shape, 2) : at::IntArrayRef(shape + 1, 1), type);
        };
        const at::Tensor token_event = get("token_event", rows, at::kInt), frame_event = get("frame_event", T, at::kInt), frame_stride = get("frame_stride", T, at::kInt),
                         event_start = get("event_start", k + 1, at::kInt), frame_offsets = get("frame_offsets", T + 1, at::kInt),
                         frame_is_key = get("frame_is_key", T, at::kByte), event_is_key = get("event_is_key", k, at::kByte),
                         frame_score = get("frame_score", T, at::kFloat), sim = get("sim", std::max<int64_t>(T - 1, 0), at::kFloat),
                         event_score = get("event_score", k, at::kFloat);
        Result r;
        r.put("sim", sim); r.put("event_start", event_start); r.put("frame_event", frame_event); r.put("out_tokens", tokens);
        r.put("frame_offsets", frame_offsets); r.put("token_event", token_event); r.put("event_is_key", event_is_key); r.put("frame_is_key", frame_is_key);
        r.put("frame_stride", frame_stride); r.put("event_score", event_score); r.put("frame_score", frame_score);
        void* stream = stream_of(a[14]);
        auto call = [&](auto... first) {
            return bound(first..., address(feats), dt, static_cast<int>(T), gh, gw, static_cast<int>(d), address(text), k, sim_mode, alpha, beta, s1, s2, reduce, edge,
                         static_cast<float*>(address(sim)), static_cast<int32_t*>(address(event_start)), static_cast<int32_t*>(address(frame_event)), address(tokens), rows, odt,
                         static_cast<int32_t*>(address(frame_offsets)), static_cast<int32_t*>(address(token_event)), static_cast<uint8_t*>(address(event_is_key)),
                         static_cast<uint8_t*>(address(frame_is_key)), static_cast<int32_t*>(address(frame_stride)), static_cast<float*>(address(event_score)),
                         static_cast<float*>(address(frame_score)), address(ws), static_cast<size_t>(ws.numel()), stream);
        };
        int rc;
        if constexpr (BATCHED) rc = launch(call(&metok_segment_compress_batched, static_cast<int>(B)));
        else rc = launch(call(&metok_segment_compress));
        return answer(rc, r);
    });
}

// ---- stage 2 -----------------------------------------------------------------------------------------------------------
// The quotas of one video, appended; returns their sum.
int64_t quotas_of(PyObject* o, std::vector<int32_t>& all) {
    need(PyList_CheckExact(o) || PyTuple_CheckExact(o));
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    PyObject** items = PySequence_Fast_ITEMS(o);
    int64_t total = 0;
    for (Py_ssize_t i = 0; i < n; ++i) { const int q = int32(items[i]); all.push_back(q); total += q; }
    return total;
}

// hidden, vis_start, n_vis, token_seg, seg_quota, q_text, k_all, token_event, event_weight, orig_idx, scores, hidden_out, workspace, out,
// score_mode, static_scratch, stream
PyObject* prefill_prune(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 17, [&](Launch& launch) -> PyObject* {
        const at::Tensor& hidden = tensor(a[0]);
        const at::Tensor& seg = tensor(a[3]);
        need(hidden.dim() == 2);
        const int64_t S = hidden.size(0), D = hidden.size(1);
        need(D <= INT32_MAX);
        const int vis_start = int32(a[1]), n_vis = int32(a[2]), mode = int32(a[14]), dt = dtype_code(hidden);
        const bool fixed = integer(a[15]) != 0;
        std::vector<int32_t> quota;
        const int64_t total = quotas_of(a[4], quota);
        const Outputs out(a[13], hidden);
        at::Tensor q, keys, scores, event, weight, orig;
        int Hq = 0, Hkv = 0, dh = 0, Tq = 0;
        if (given(a[5])) {
            q = tensor(a[5]); keys = tensor(a[6]);
            need(q.dim() == 3 && keys.dim() == 3 && keys.size(1) == S && keys.size(2) == q.size(2) && dtype_code(q) == dt && dtype_code(keys) == dt);
            for (int i = 0; i < 3; ++i) need(q.size(i) <= INT32_MAX && keys.size(i) <= INT32_MAX);
            Hq = static_cast<int>(q.size(0)); Tq = static_cast<int>(q.size(1)); dh = static_cast<int>(q.size(2)); Hkv = static_cast<int>(keys.size(0));
            scores = out.get("scores", {n_vis}, at::kFloat);
        } else {
            need(!given(a[6]));
            scores = tensor(a[10]);
        }
        if (given(a[7])) event = tensor(a[7]);
        if (given(a[8])) weight = tensor(a[8]);
        if (given(a[9])) orig = tensor(a[9]);
        at::Tensor ws;
        if (!fixed) ws = workspace_of(a[12], out, given(a[12]) ? 0 : metok_prefill_prune_workspace_bytes(S, Hq, Hkv, dh, Tq, n_vis, dt));
        const at::Tensor kept = out.get("kept_idx", {total}, at::kInt), seg_out = out.get("token_seg_out", {total}, at::kInt), orig_out = out.get("orig_idx_out", {total}, at::kInt);
        at::Tensor event_out;
        if (event.defined()) event_out = out.get("token_event_out", {total}, at::kInt);
        const int64_t rows = S - n_vis + total;
        at::Tensor hidden_out;
        PyObject* ho = given(a[11]) ? a[11] : out.find("hidden_out");
        if (ho) {
            hidden_out = tensor(ho);
            need(hidden_out.dim() == 2 && hidden_out.size(0) == rows && hidden_out.size(1) == D && hidden_out.scalar_type() == hidden.scalar_type());
        } else {
            hidden_out = out.fresh({rows, D}, hidden.scalar_type());
        }
        auto at_ = [](const at::Tensor& t) -> void* { return t.defined() ? address(t) : nullptr; };
        const int n_events = weight.defined() ? static_cast<int>(weight.numel()) : 0;
        Result r;
        r.put("scores", scores); r.put("kept_idx", kept);
        if (ho) { Py_INCREF(ho); r.put("hidden_out", ho); } else r.put("hidden_out", hidden_out);
        r.put("token_seg_out", seg_out); r.put("orig_idx_out", orig_out);
        if (event_out.defined()) r.put("token_event_out", event_out);
        void* stream = stream_of(a[16]);
        auto call = [&](auto f, auto... last) {
            return bound(f, address(hidden), S, static_cast<int>(D), dt, at_(q), at_(keys), Hq, Hkv, dh, Tq, mode, vis_start, n_vis, static_cast<const int32_t*>(address(seg)),
                         static_cast<const int32_t*>(at_(event)), static_cast<const float*>(at_(weight)), n_events, static_cast<int>(quota.size()), quota.data(),
                         static_cast<const int32_t*>(at_(orig)), static_cast<float*>(address(scores)), static_cast<int32_t*>(address(kept)), address(hidden_out),
                         static_cast<int32_t*>(address(seg_out)), static_cast<int32_t*>(at_(event_out)), static_cast<int32_t*>(address(orig_out)), last...);
        };
        return answer(fixed ? launch(call(&metok_prefill_prune_static, stream))
                            : launch(call(&metok_prefill_prune, address(ws), static_cast<size_t>(ws.numel()), stream)), r);
    });
}

// hidden, vis_start, n_vis, token_seg, seg_quota, q_text, k_all, token_event, event_weight, orig_idx, scores, hidden_out, workspace, out,
// score_mode, keep_stride, out_row_stride, stream
PyObject* prefill_prune_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 18, [&](Launch& launch) -> PyObject* {
        const at::Tensor& hidden = tensor(a[0]);
        const at::Tensor& seg = tensor(a[3]);
        need(hidden.dim() == 3);
        const int64_t B = hidden.size(0), S = hidden.size(1), D = hidden.size(2);
        need(B >= 1 && B <= METOK_MAX_BATCH && D <= INT32_MAX);
        const int vis_start = int32(a[1]), n_vis = int32(a[2]), mode = int32(a[14]), dt = dtype_code(hidden);
        need(PyList_CheckExact(a[4]) || PyTuple_CheckExact(a[4]));
        need(PySequence_Fast_GET_SIZE(a[4]) == B);
        std::vector<int32_t> quota;
        std::vector<int64_t> keep;
        int64_t most = 0;
        for (int64_t b = 0; b < B; ++b) {
            keep.push_back(quotas_of(PySequence_Fast_ITEMS(a[4])[b], quota));
            most = b ? std::max(most, keep[b]) : keep[0];
        }
        const int n_seg = static_cast<int>(quota.size() / B);
        for (int64_t b = 0; b < B; ++b) need(PySequence_Fast_GET_SIZE(PySequence_Fast_ITEMS(a[4])[b]) == n_seg);
        const Outputs out(a[13], hidden);
        auto is = [](const at::Tensor& t, int64_t r, int64_t c) { return t.dim() == 2 && t.size(0) == r && t.size(1) == c; };
        at::Tensor q, keys, scores, event, weight, orig;
        int Hq = 0, Hkv = 0, dh = 0, Tq = 0;
        if (given(a[5])) {
            q = tensor(a[5]); keys = tensor(a[6]);
            need(q.dim() == 4 && keys.dim() == 4 && q.size(0) == B && keys.size(0) == B && keys.size(2) == S && keys.size(3) == q.size(3) && dtype_code(q) == dt && dtype_code(keys) == dt);
            for (int i = 0; i < 4; ++i) need(q.size(i) <= INT32_MAX && keys.size(i) <= INT32_MAX);
            Hq = static_cast<int>(q.size(1)); Tq = static_cast<int>(q.size(2)); dh = static_cast<int>(q.size(3)); Hkv = static_cast<int>(keys.size(1));
            scores = out.get("scores", {B, n_vis}, at::kFloat);
        } else {
            need(!given(a[6]));
            scores = tensor(a[10]);
            need(is(scores, B, n_vis));
        }
        need(is(seg, B, n_vis));
        if (given(a[7])) { event = tensor(a[7]); need(is(event, B, n_vis)); }
        if (given(a[8])) { weight = tensor(a[8]); need(weight.dim() == 2 && weight.size(0) == B && weight.size(1) <= INT32_MAX); }
        if (given(a[9])) { orig = tensor(a[9]); need(orig.dim() == 2 && orig.size(0) == B && orig.size(1) >= n_vis); }
        const at::Tensor ws = workspace_of(a[12], out, given(a[12]) ? 0 : metok_prefill_prune_batched_workspace_bytes(static_cast<int>(B), S, Hq, Hkv, dh, Tq, n_vis, dt));
        const bool in_place = a[11] == a[0];
        const int64_t keep_stride = given(a[15]) ? integer(a[15]) : most;
        const int64_t row_stride = given(a[16]) ? integer(a[16]) : (in_place ? S : S - n_vis + most);
        const at::Tensor kept = out.get("kept_idx", {B, keep_stride}, at::kInt);
        at::Tensor hidden_out;
        PyObject* ho = given(a[11]) ? a[11] : out.find("hidden_out");
        if (ho) {
            hidden_out = tensor(ho);
            need(hidden_out.dim() == 3 && hidden_out.size(0) == B && hidden_out.size(1) == row_stride && hidden_out.size(2) == D && hidden_out.scalar_type() == hidden.scalar_type());
        } else {
            hidden_out = out.fresh({B, row_stride, D}, hidden.scalar_type());
        }
        const at::Tensor seg_out = out.get("token_seg_out", {B, keep_stride}, at::kInt);
        at::Tensor event_out, orig_out;
        if (event.defined()) event_out = out.get("token_event_out", {B, keep_stride}, at::kInt);
        if (PyObject* v = out.find("orig_idx_out")) {              // may be wider than the other lists
            orig_out = tensor(v);
            need(orig_out.scalar_type() == at::kInt && orig_out.dim() == 2 && orig_out.size(0) == B);
        } else {
            orig_out = out.fresh({B, keep_stride}, at::kInt);
        }
        auto at_ = [](const at::Tensor& t) -> void* { return t.defined() ? address(t) : nullptr; };
        Result r;
        r.put("scores", scores); r.put("kept_idx", kept);
        if (ho) { Py_INCREF(ho); r.put("hidden_out", ho); } else r.put("hidden_out", hidden_out);
        r.put("token_seg_out", seg_out); r.put("orig_idx_out", orig_out);
        Owned list(PyList_New(static_cast<Py_ssize_t>(B)));
        for (int64_t b = 0; b < B; ++b) PyList_SET_ITEM(list.o, b, Owned(PyLong_FromLongLong(keep[b])).release());
        r.put("n_keep", list.release());
        if (event_out.defined()) r.put("token_event_out", event_out);
        void* stream = stream_of(a[17]);
        return answer(launch(bound(&metok_prefill_prune_batched, static_cast<int>(B), address(hidden), S, static_cast<int>(D), dt, at_(q), at_(keys), Hq, Hkv, dh, Tq, mode,
                                   vis_start, n_vis, static_cast<const int32_t*>(address(seg)), static_cast<const int32_t*>(at_(event)), static_cast<const float*>(at_(weight)),
                                   weight.defined() ? static_cast<int>(weight.size(1)) : 0, n_seg, quota.data(), static_cast<const int32_t*>(at_(orig)),
                                   orig.defined() ? orig.size(1) : int64_t{0}, static_cast<float*>(address(scores)), static_cast<int32_t*>(address(kept)), keep_stride,
                                   address(hidden_out), row_stride, static_cast<int32_t*>(address(seg_out)), static_cast<int32_t*>(at_(event_out)),
                                   static_cast<int32_t*>(address(orig_out)), orig_out.size(1), address(ws), static_cast<size_t>(ws.numel()), stream)), r);
    });
}

// ---- stage 3 -----------------------------------------------------------------------------------------------------------
// The per-layer buffers (all of the first one's shape) and index lists of a cache.
struct Layers {
    std::vector<void*> k, v;
    std::vector<const int32_t*> idx;
    std::vector<int32_t> n_keep;
    at::Tensor first;
    int L = 0, dt = 0;

    Layers(PyObject* ks, PyObject* vs) {
        need((PyList_CheckExact(ks) || PyTuple_CheckExact(ks)) && (PyList_CheckExact(vs) || PyTuple_CheckExact(vs)));
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(ks);
        need(n >= 1 && n <= METOK_MAX_LAYERS && PySequence_Fast_GET_SIZE(vs) == n);
        L = static_cast<int>(n);
        first = tensor(PySequence_Fast_ITEMS(ks)[0]);
        need(first.dim() == 4);
        for (int i = 0; i < 4; ++i) need(first.size(i) <= INT32_MAX);
        dt = dtype_code(first);
        for (int side = 0; side < 2; ++side) {
            PyObject** items = PySequence_Fast_ITEMS(side ? vs : ks);
            for (int l = 0; l < L; ++l) {
                const at::Tensor& t = tensor(items[l]);
                need(t.sizes() == first.sizes());
                (side ? v : k).push_back(address(t));
            }
        }
    }
    void lists(PyObject* o, int64_t B) {
        need((PyList_CheckExact(o) || PyTuple_CheckExact(o)) && PySequence_Fast_GET_SIZE(o) == L);
        for (int l = 0; l < L; ++l) {
            PyObject* e = PySequence_Fast_ITEMS(o)[l];
            if (!given(e)) { idx.push_back(nullptr); n_keep.push_back(0); continue; }
            const at::Tensor& t = tensor(e);
            need(t.scalar_type() == at::kInt && t.dim() == 2 && t.size(0) == B && t.numel() > 0 && t.size(1) <= INT32_MAX);
            idx.push_back(static_cast<const int32_t*>(address(t)));
            n_keep.push_back(static_cast<int32_t>(t.size(1)));
        }
    }
};

// k_layers, v_layers, page_table (None: dense), idx, new_len, workspace, stream
PyObject* kv_compact(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 7, [&](Launch& launch) -> PyObject* {
        Layers x(a[0], a[1]);
        const bool paged = given(a[2]);
        at::Tensor table;
        if (paged) {
            table = tensor(a[2]);
            need(table.scalar_type() == at::kInt && table.dim() == 2 && table.size(0) <= INT32_MAX && table.size(1) <= INT32_MAX);
        }
        const int64_t B = paged ? table.size(0) : x.first.size(0), Hkv = x.first.size(1), rows = x.first.size(2), dh = x.first.size(3);
        x.lists(a[3], B);
        const Outputs out(Py_None, x.first);
        at::Tensor len = given(a[4]) ? tensor(a[4]) : out.fresh({x.L}, at::kInt);
        const int64_t cap = paged ? table.size(1) * rows : rows;
        const at::Tensor ws = workspace_of(a[5], out, given(a[5]) ? 0 : metok_kv_compact_workspace_bytes(x.L, static_cast<int>(B), static_cast<int>(Hkv), cap, static_cast<int>(dh), x.dt));
        if (given(a[4])) Py_INCREF(a[4]);
        Owned result(given(a[4]) ? a[4] : THPVariable_Wrap(len));
        void* stream = stream_of(a[6]);
        auto call = [&](auto f, auto... middle) {
            return bound(f, x.k.data(), x.v.data(), x.L, static_cast<int>(B), static_cast<int>(Hkv), middle..., x.idx.data(), x.n_keep.data(),
                         static_cast<int32_t*>(address(len)), address(ws), static_cast<size_t>(ws.numel()), stream);
        };
        return answer(paged ? launch(call(&metok_kv_compact_paged, x.first.size(0), static_cast<int>(rows), static_cast<int>(dh), x.dt,
                                          static_cast<const int32_t*>(address(table)), static_cast<int>(table.size(1))))
                            : launch(call(&metok_kv_compact, rows, static_cast<int>(dh), x.dt)), result);
    });
}

// k_pools, v_pools, page_table, idx, len_in, workspace, stream
PyObject* kv_relink_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded(n, 7, [&](Launch& launch) -> PyObject* {
        Layers x(a[0], a[1]);
        const at::Tensor& table = tensor(a[2]);
        need(table.scalar_type() == at::kInt && (table.dim() == 2 || (table.dim() == 3 && table.size(0) == x.L)));
        const int64_t B = table.size(-2), pages = table.size(-1), L = x.L;
        need(B <= INT32_MAX && pages <= INT32_MAX);
        x.lists(a[3], B);
        std::vector<int32_t> lens;
        if (given(a[4])) {
            quotas_of(a[4], lens);
            need(static_cast<int64_t>(lens.size()) == L);
        }
        const Outputs out(Py_None, x.first);
        const at::Tensor table_out = out.fresh({L, B, pages}, at::kInt), free_pages = out.fresh({L, B, pages}, at::kInt), n_free = out.fresh({L, B}, at::kInt),
                         copied = out.fresh({L, B}, at::kInt), len = out.fresh({L}, at::kInt);
        const int Hkv = static_cast<int>(x.first.size(1)), ps = static_cast<int>(x.first.size(2)), dh = static_cast<int>(x.first.size(3));
        const at::Tensor ws = workspace_of(a[5], out, given(a[5]) ? 0 : metok_kv_relink_paged_workspace_bytes(x.L, static_cast<int>(B), Hkv, ps, static_cast<int>(pages), dh, x.dt));
        Result r;
        r.put("page_table_out", table_out); r.put("free_pages", free_pages); r.put("n_free", n_free); r.put("rows_copied", copied); r.put("new_len", len);
        if (given(a[5])) { Py_INCREF(a[5]); r.put("workspace", a[5]); } else r.put("workspace", ws);
        void* stream = stream_of(a[6]);
        return answer(launch(bound(&metok_kv_relink_paged, x.k.data(), x.v.data(), x.L, static_cast<int>(B), Hkv, x.first.size(0), ps, dh, x.dt,
                                   static_cast<const int32_t*>(address(table)), table.dim() == 2 ? int64_t{0} : B * pages, static_cast<int>(pages),
                                   given(a[4]) ? lens.data() : nullptr, x.idx.data(), x.n_keep.data(), static_cast<int32_t*>(address(table_out)),
                                   static_cast<int32_t*>(address(free_pages)), static_cast<int32_t*>(address(n_free)), static_cast<int32_t*>(address(copied)),
                                   static_cast<int32_t*>(address(len)), address(ws), static_cast<size_t>(ws.numel()), stream)), r);
    });
}

#define METOK_HOST_CALL(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr
PyMethodDef methods[] = {
    {"segment_compress", METOK_HOST_CALL(&segment_compress<false>)},
    {"segment_compress_batched", METOK_HOST_CALL(&segment_compress<true>)},
    {"prefill_prune", METOK_HOST_CALL(&prefill_prune)},
    {"prefill_prune_batched", METOK_HOST_CALL(&prefill_prune_batched)},
    {"kv_compact", METOK_HOST_CALL(&kv_compact)},
    {"kv_relink_paged", METOK_HOST_CALL(&kv_relink_paged)},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The tensors' layout is that of the torch whose headers this was built with.
PyMODINIT_FUNC PyInit__host() {
    try {
        const Owned torch(PyImport_ImportModule("torch")), version(PyObject_GetAttrString(torch.o, "__version__"));
        const Owned text(PyObject_Str(version.o));
        if (PyUnicode_CompareWithASCIIString(text.o, METOK_TORCH_VERSION) != 0) {
            PyErr_Format(PyExc_ImportError, "built for torch %s, this is %U", METOK_TORCH_VERSION, text.o);
            return nullptr;
        }
    } catch (const Raised&) {
        return nullptr;
    }
    return PyModule_Create(&module);
}
