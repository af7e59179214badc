// Argument marshalling of the serving calls (mla.py) in native code.
//
// A decode step is three calls whose kernels together take 14 to 20 us at small sizes; checking the tensors,
// asking for the stream and converting some twenty arguments each in Python took 6 to 8 us per call, so that
// the host set the pace below about 25 us per step.  The functions here read the tensors' fields directly and
// call the C entry point they are given.  They accept what mla.py's checks let through, as far as it is plain torch
// tensors, integers and floats: inputs of the expected types and shapes, tables of int32, and outputs of the
// expected element size with room for the result (their own shape and type are the caller's).  For anything else
// they return None without having called anything, and mla.py goes through its own checks, which raise.
// No arithmetic, no allocation, no state beyond the entry points' addresses; the interpreter lock is released
// around the call as ctypes does.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include "mla_gfx950.h"

namespace {

decltype(&mla_absorb_q) p_absorb_q;
decltype(&mla_out_proj) p_out_proj;
decltype(&mla_decode_paged_multi) p_decode;
decltype(&mla_merge_out_proj_multi) p_merge_out_proj;
decltype(&mla_merge_partials) p_merge_partials;
decltype(&mla_cache_append) p_append;

struct No {};   // the arguments are not of the plain kind

// a contiguous tensor on the GPU
const at::Tensor& tensor(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) throw No();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) throw No();
    return t;
}

long integer(PyObject* o)
{
    if (!PyLong_CheckExact(o)) throw No();
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) throw No();
    return v;
}
float real(PyObject* o)
{
    if (!PyFloat_CheckExact(o)) throw No();
    return (float)PyFloat_AS_DOUBLE(o);
}
int dim(int64_t v)
{
    if (v > INT32_MAX) throw No();
    return (int)v;
}
mla_dtype io_type(const at::Tensor& t)
{
    if (t.scalar_type() == at::kFloat) return MLA_F32;
    if (t.scalar_type() == at::kBFloat16) return MLA_BF16;
    throw No();
}
mla_dtype cache_type(const at::Tensor& t)
{
    if (t.scalar_type() == at::kByte || t.scalar_type() == at::kFloat8_e4m3fn) return MLA_FP8_E4M3;
    return io_type(t);
}
void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }
void require(bool ok)
{
    if (!ok) throw No();
}

// an output (or scratch) with room for n elements of `size` bytes
void* room(PyObject* o, int64_t n, size_t size)
{
    const at::Tensor& t = tensor(o);
    require((size_t)t.element_size() == size && t.numel() >= n);
    return t.data_ptr();
}
void* room_or_null(PyObject* o, int64_t n, size_t size) { return o == Py_None ? nullptr : room(o, n, size); }
size_t size_of(mla_dtype io) { return io == MLA_F32 ? 4 : 2; }

// f(): the status of the call it makes
template <typename F> PyObject* guarded(F f)
{
    try {
        return PyLong_FromLong(f());
    } catch (...) {       // No, or what a tensor without storage throws: the caller's own checks find it again
        Py_RETURN_NONE;
    }
}
template <typename F> int unlocked(F f)
{
    PyThreadState* s = PyEval_SaveThread();
    const int r = f();
    PyEval_RestoreThread(s);
    return r;
}

// (x [B, H, K], W [H, K, N], out)
template <typename P> PyObject* projection(P p, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&] {
        require(n == 3);
        const at::Tensor &x = tensor(a[0]), &W = tensor(a[1]);
        require(x.dim() == 3 && W.dim() == 3 && W.size(0) == x.size(1) && W.size(1) == x.size(2) && W.scalar_type() == x.scalar_type());
        const int B = dim(x.size(0)), H = dim(x.size(1)), K = dim(x.size(2)), N = dim(W.size(2));
        const mla_dtype io = io_type(x);
        void *px = x.data_ptr(), *pw = W.data_ptr(), *po = room(a[2], (int64_t)B * H * N, size_of(io)), *s = stream_of(x);
        return unlocked([&] { return p(px, pw, po, B, H, K, N, io, s); });
    });
}
PyObject* absorb_q(PyObject*, PyObject* const* a, Py_ssize_t n) { return projection(p_absorb_q, a, n); }
PyObject* out_proj(PyObject*, PyObject* const* a, Py_ssize_t n) { return projection(p_out_proj, a, n); }

// (dimensions of q_abs, q_abs, q_rope | None, kv_cache, page_table, seq_lens, scale, num_splits, kv_scale | None, workspace,
//  out | None, lse | None, flags); q_abs [B, H, d_c] or [B, T, H, d_c]
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&] {
        require(n == 13);
        const int k = (int)integer(*a++);
        const at::Tensor &q = tensor(a[0]), &kv = tensor(a[2]), &table = tensor(a[3]), &lens = tensor(a[4]), &ws = tensor(a[8]);
        require((k == 3 || k == 4) && q.dim() == k && kv.dim() == 3);
        const int64_t B = q.size(0), T = k == 4 ? q.size(1) : 1, H = q.size(k - 2), d_c = q.size(k - 1);
        const int64_t pages = kv.size(0), page = kv.size(1), d_rope = kv.size(2) - d_c;
        require(d_rope >= 0);
        void* pr = nullptr;
        if (a[1] != Py_None) {
            const at::Tensor& r = tensor(a[1]);
            if (d_rope) {
                require(r.dim() == k && r.size(0) == B && r.size(k - 2) == H && r.size(k - 1) == d_rope && (k == 3 || r.size(1) == T) &&
                        r.scalar_type() == q.scalar_type());
            }
            pr = r.data_ptr();
        } else {
            require(d_rope == 0);
        }
        require(table.scalar_type() == at::kInt && lens.scalar_type() == at::kInt && table.dim() == 2 && table.size(0) == B &&
                lens.dim() == 1 && lens.size(0) == B);
        const float* ps = nullptr;
        if (a[7] != Py_None) {
            const at::Tensor& s = tensor(a[7]);
            require(s.scalar_type() == at::kFloat && s.dim() == 2 && s.size(0) == pages && s.size(1) == page);
            ps = static_cast<const float*>(s.data_ptr());
        }
        const mla_dtype io = io_type(q), cache = cache_type(kv);
        void *pq = q.data_ptr(), *pkv = kv.data_ptr(), *pws = ws.data_ptr();
        void *po = room_or_null(a[9], q.numel(), size_of(io)), *pl = room_or_null(a[10], B * T * H, 4);
        const auto* pt = static_cast<const int32_t*>(table.data_ptr());
        const auto* pn = static_cast<const int32_t*>(lens.data_ptr());
        const size_t bytes = ws.nbytes();
        const float scale = real(a[5]);
        const int splits = (int)integer(a[6]), flags = (int)integer(a[11]);
        const int b = dim(B), t = dim(T), h = dim(H), dc = dim(d_c), dr = dim(d_rope), pg = dim(page), np = dim(pages), mp = dim(table.size(1));
        void* s = stream_of(q);
        return unlocked([&] {
            return p_decode(pq, pr, pkv, ps, pt, pn, po, static_cast<float*>(pl), pws, bytes, b, t, h, dc, dr, pg, np, mp, splits, scale, io,
                            cache, (unsigned)flags, s);
        });
    });
}

// (workspace, W_UV, o_lat, lse | None, out, B, q_len, num_splits, flags)
PyObject* merge_out_proj(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&] {
        require(n == 9);
        const at::Tensor &ws = tensor(a[0]), &W = tensor(a[1]);
        require(W.dim() == 3);
        const int B = (int)integer(a[5]), T = (int)integer(a[6]), S = (int)integer(a[7]), flags = (int)integer(a[8]);
        const int H = dim(W.size(0)), d_c = dim(W.size(1)), d_head = dim(W.size(2));
        const mla_dtype io = io_type(W);
        require(B >= 0 && B <= 65535 && T >= 0 && T <= 65535 && (int64_t)B * T <= 65535 && H <= 65535);   // (no more is taken: the products below fit)
        const int64_t rows = (int64_t)B * T * H;
        void *pws = ws.data_ptr(), *pw = W.data_ptr(), *po = room(a[2], rows * d_c, size_of(io)), *pl = room_or_null(a[3], rows, 4),
             *pout = room(a[4], rows * d_head, size_of(io));
        const size_t bytes = ws.nbytes();
        void* s = stream_of(ws);
        return unlocked([&] {
            return p_merge_out_proj(pws, bytes, pw, po, static_cast<float*>(pl), pout, B, T, H, d_c, d_head, S, io, (unsigned)flags, s);
        });
    });
}

// (workspace, out, lse | None, B, H, d_c, num_splits, flags)
PyObject* merge_partials(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&] {
        require(n == 8);
        const at::Tensor &ws = tensor(a[0]), &out = tensor(a[1]);
        const int B = (int)integer(a[3]), H = (int)integer(a[4]), d_c = (int)integer(a[5]), S = (int)integer(a[6]), flags = (int)integer(a[7]);
        const mla_dtype io = io_type(out);
        require(B >= 0 && B <= 65535 && H >= 0 && H <= 65535 && d_c >= 0);
        void *pws = ws.data_ptr(), *po = room(a[1], (int64_t)B * H * d_c, size_of(io)), *pl = room_or_null(a[2], (int64_t)B * H, 4);
        const size_t bytes = ws.nbytes();
        void* s = stream_of(ws);
        return unlocked([&] { return p_merge_partials(pws, bytes, po, static_cast<float*>(pl), B, H, d_c, S, io, (unsigned)flags, s); });
    });
}

// (x, W_DKVR, kv_cache, kv_scale | None, page_table, positions, workspace, d_c, rope_base)
PyObject* cache_append(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded([&] {
        require(n == 9);
        const at::Tensor &x = tensor(a[0]), &W = tensor(a[1]), &kv = tensor(a[2]), &table = tensor(a[4]), &pos = tensor(a[5]), &ws = tensor(a[6]);
        require(x.dim() == 2 && W.dim() == 2 && kv.dim() == 3 && table.dim() == 2);
        require(W.size(0) == x.size(1) && W.size(1) == kv.size(2) && W.scalar_type() == x.scalar_type());
        require(table.scalar_type() == at::kInt && table.size(0) >= x.size(0) && pos.scalar_type() == at::kInt && pos.numel() >= x.size(0));
        const int d_c = (int)integer(a[7]);
        void *px = x.data_ptr(), *pw = W.data_ptr(), *pkv = kv.data_ptr(), *ps = room_or_null(a[3], kv.size(0) * kv.size(1), 4),
             *pws = ws.data_ptr();
        const auto* pt = static_cast<const int32_t*>(table.data_ptr());
        const auto* pp = static_cast<const int32_t*>(pos.data_ptr());
        const int B = dim(x.size(0)), D = dim(x.size(1)), d_rope = dim(W.size(1)) - d_c, page = dim(kv.size(1)), pages = dim(kv.size(0)),
                  mp = dim(table.size(1));
        const float base = real(a[8]);
        const mla_dtype io = io_type(x), cache = cache_type(kv);
        const size_t bytes = (size_t)ws.numel();
        void* s = stream_of(x);
        return unlocked([&] {
            return p_append(px, pw, pkv, static_cast<float*>(ps), pt, pp, pws, bytes, B, D, d_c, d_rope, page, pages, mp, base, io, cache, s);
        });
    });
}

// (addresses of the six entry points, in the order above)
PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long p[6];
    if (!PyArg_ParseTuple(args, "KKKKKK", p, p + 1, p + 2, p + 3, p + 4, p + 5)) return nullptr;
    p_absorb_q = reinterpret_cast<decltype(p_absorb_q)>(p[0]);
    p_out_proj = reinterpret_cast<decltype(p_out_proj)>(p[1]);
    p_decode = reinterpret_cast<decltype(p_decode)>(p[2]);
    p_merge_out_proj = reinterpret_cast<decltype(p_merge_out_proj)>(p[3]);
    p_merge_partials = reinterpret_cast<decltype(p_merge_partials)>(p[4]);
    p_append = reinterpret_cast<decltype(p_append)>(p[5]);
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(absorb_q), FAST(out_proj), FAST(decode), FAST(merge_out_proj), FAST(merge_partials), FAST(cache_append),
                         {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module_def); }
