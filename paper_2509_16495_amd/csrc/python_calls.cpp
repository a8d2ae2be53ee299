// The Python binding's calls (binding.py), natively: arguments are checked and turned into those of the C ABI here, so that a
// small call costs the host little more than its launches.  What a call spent in Python - shapes and strides asked one by one,
// a ctypes structure filled, nineteen ctypes arguments converted - was 2.2 us for an exchange and 4.8 us for an attention call,
// a third of the whole call where there is little to compute.  Here it is 0.3 and 0.4.
//
// The functions take what binding.py's take, positionally and complete, and return the library's status; what is refused is
// refused with the same exceptions.  They hold no state but the library's addresses and the allocator (bind()).
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "shiftattn.h"

namespace {

// the library's functions: one list for the pointers, the names that binding.py looks them up by, and their order in bind()
#define SHIFTATTN_FUNCTIONS(F)                                                                                         \
    F(pack, pack_seq2head) F(unpack, unpack_head2seq) F(prefill, prefill) F(decode, decode) F(decode_static, decode_static) \
    F(mixed, mixed) F(kv_write, kv_write) F(qkv, qkv_proj_pack_ws) F(o_proj, unpack_o_proj_ws) F(qkv_plain, qkv_proj_pack)   \
    F(o_proj_plain, unpack_o_proj) F(qkv_fp8, qkv_proj_pack_fp8_ws) F(o_proj_fp8, unpack_o_proj_fp8_ws)                      \
    F(quantize_rows, quantize_rows_fp8) F(quantize_recv, quantize_recv_fp8)                                                 \
    F(prefill_bytes, prefill_workspace_bytes) F(decode_bytes, decode_workspace_bytes) F(mixed_bytes, mixed_workspace_bytes)
struct Library {
#define SHIFTATTN_POINTER(member, name) decltype(&shiftattn_##name) member;
    SHIFTATTN_FUNCTIONS(SHIFTATTN_POINTER)
};
#define SHIFTATTN_NAME(member, name) "shiftattn_" #name,
constexpr const char* kNames[] = {SHIFTATTN_FUNCTIONS(SHIFTATTN_NAME)};
constexpr Py_ssize_t kFunctions = sizeof(Library) / sizeof(void*);
Library lib{};
PyObject* allocate = nullptr;   // binding.py's: (bytes, tensor on the device wanted) -> tensor

struct Refused {
    PyObject* type;
    std::string what;
};
struct PythonError {};   // already set

void need(bool ok, const char* what) {
    if (!ok) throw Refused{PyExc_AssertionError, what};
}
const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) throw Refused{PyExc_TypeError, std::string("a torch.Tensor is wanted, not ") + Py_TYPE(o)->tp_name};
    return THPVariable_Unpack(o);
}
const at::Tensor* tensor_or_none(PyObject* o) { return o == Py_None ? nullptr : &tensor(o); }
// (the last check of an argument: kernels reach device memory and pinned host memory, an empty tensor has none)
void* ptr(const at::Tensor& t) {
    if (!t.is_cuda() && t.numel() != 0 && !(t.device().is_cpu() && t.is_pinned()))
        throw Refused{PyExc_RuntimeError, "a tensor on the GPU is wanted, not on " + t.device().str()};
    return t.data_ptr();
}
void* ptr(const at::Tensor* t) { return t ? ptr(*t) : nullptr; }
// a workspace: its bytes in one piece
const at::Tensor& dense(const at::Tensor& t) {
    need(t.is_non_overlapping_and_dense(), "workspace: without gaps or overlaps");
    return t;
}
const at::Tensor* dense_or_none(PyObject* o) { return o == Py_None ? nullptr : &dense(tensor(o)); }
size_t bytes(const at::Tensor* t) { return t ? t->nbytes() : 0; }
// (as ctypes takes them: anything with __index__ / __float__, whole numbers cut to 32 bits)
int32_t whole(PyObject* o) {
    const unsigned long v = PyLong_AsUnsignedLongMask(o);
    if (v == static_cast<unsigned long>(-1) && PyErr_Occurred()) throw PythonError{};
    return static_cast<int32_t>(v);
}
float real(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PythonError{};
    return static_cast<float>(v);
}
void dims(const at::Tensor& t, int64_t n, const char* name) {
    if (t.dim() != n) throw Refused{PyExc_ValueError, std::string(name) + ": " + std::to_string(n) + " dimensions wanted, not " + std::to_string(t.dim())};
}
int32_t dtype_code(const at::Tensor& t) {
    if (t.scalar_type() == at::kBFloat16) return SHIFTATTN_BF16;
    if (t.scalar_type() == at::kFloat) return SHIFTATTN_F32;
    throw Refused{PyExc_TypeError, std::string("unsupported tensor dtype ") + c10::toString(t.scalar_type())};
}
int32_t cut(int64_t v) { return static_cast<int32_t>(v); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// elements between consecutive tokens of a [tokens, heads, D] view whose inner two dims are dense
int64_t row_stride(const at::Tensor& t) {
    const auto shape = t.sizes(), stride = t.strides();
    need(shape.size() == 3 && stride[2] == 1 && (shape[1] == 1 || stride[1] == shape[2]), "inner dims must be dense");
    return shape[0] > 1 ? stride[0] : shape[1] * shape[2];
}

shiftattn_xchg exchange(int64_t P, int64_t h, int64_t h_kv, int64_t D, int32_t dtype) {
    shiftattn_xchg x{};
    x.P = cut(P), x.num_q_heads = cut(h), x.num_kv_heads = cut(h_kv), x.head_dim = cut(D), x.dtype = dtype;
    return x;
}
int64_t local_kv_heads(int64_t P, int64_t h_kv) { return h_kv == 0 ? 0 : h_kv >= P ? h_kv / P : 1; }

constexpr int64_t kBlock = 16;

shiftattn_attn describe(const at::Tensor& q, const at::Tensor& cache, const at::Tensor& table, PyObject* scale, const at::Tensor* k_new,
                        const at::Tensor* out, PyObject* k_scale, PyObject* v_scale) {
    dims(q, 3, "q");
    dims(cache, 4, "kv_cache");
    const bool fp8 = cache.scalar_type() == at::kByte;
    need(cache.size(2) == 2 && cache.size(3) == kBlock * q.size(2) && cache.is_contiguous() && (fp8 || cache.scalar_type() == q.scalar_type()),
         "kv_cache: contiguous [num_blocks, hkv_l, 2, 16 * D] of q's type or uint8");
    need(table.scalar_type() == at::kInt && table.dim() == 2 && table.is_contiguous(), "block_table: contiguous int32 [num_seqs, max_blocks]");
    shiftattn_attn a{};
    a.num_q_heads = cut(q.size(1)), a.num_kv_heads = cut(cache.size(1)), a.head_dim = cut(q.size(2)), a.dtype = dtype_code(q);
    a.block_size = kBlock, a.num_blocks = cut(cache.size(0)), a.max_blocks_per_seq = cut(table.size(1));
    a.softmax_scale = real(scale);
    a.q_stride = row_stride(q), a.kv_stride = k_new ? row_stride(*k_new) : 0, a.out_stride = out ? row_stride(*out) : 0;
    a.kv_format = fp8 ? SHIFTATTN_KV_FP8_E4M3 : SHIFTATTN_KV_SAME;
    a.k_scale = real(k_scale), a.v_scale = real(v_scale);
    return a;
}

// The workspace of a call: what it brings, else what the library asks for, allocated once the arguments have passed.  Where the
// library has no size for them it refuses them, so that call goes ahead without one and names the reason.
struct Owned {
    PyObject* object = nullptr;
    ~Owned() { Py_XDECREF(object); }
};
template <class Bytes>
const at::Tensor* workspace(PyObject* given, PyObject* like, Owned& own, Bytes wanted) {
    if (given != Py_None) return &dense(tensor(given));
    ptr(tensor(like));   // (nothing is allocated for host tensors)
    const size_t n = wanted();
    if (n == 0 || n == SIZE_MAX) return nullptr;
    own.object = PyObject_CallFunction(allocate, "KO", static_cast<unsigned long long>(n), like);
    if (!own.object) throw PythonError{};
    return &tensor(own.object);
}

// rows that share memory: their stride of 0 would stand for dense rows in the library
void apart(const at::Tensor& t) { need(t.size(0) <= 1 || t.stride(0) > 0, "rows must not share memory"); }
// the rows that a call reads and writes, and those that it appends to the cache where it brings all three tensors of them (the
// library refuses one or two)
void rows_of(const at::Tensor& q, const at::Tensor& out, const at::Tensor* k, const at::Tensor* v, const at::Tensor* slots, const at::Tensor& cache) {
    apart(q);
    apart(out);
    if (!k || !v || !slots) return;
    apart(*k);
    dims(*k, 3, "k_new");
    need(k->size(0) >= q.size(0) && k->size(1) == cache.size(1) && k->size(2) == q.size(2) && k->scalar_type() == q.scalar_type(),
         "k_new: [a row per row of q, hkv_l, D] of its type");
    need(v->sizes() == k->sizes() && v->scalar_type() == k->scalar_type() && row_stride(*v) == row_stride(*k), "v_new: shape, type and row stride of k_new");
    need(slots->scalar_type() == at::kLong && slots->size(0) >= q.size(0) && slots->is_contiguous(), "slot_mapping: contiguous int64, one per row of q");
}

// body() checks and returns the call to make, which runs without the interpreter's lock, as through ctypes
template <class Body>
PyObject* run(Py_ssize_t given, Py_ssize_t wanted, Body body) {
    if (given != wanted) {
        PyErr_Format(PyExc_TypeError, "%zd arguments wanted, not %zd", wanted, given);
        return nullptr;
    }
    try {
        const auto call = body();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = call();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    } catch (const Refused& r) {
        PyErr_SetString(r.type, r.what.c_str());
    } catch (const PythonError&) {
    } catch (const c10::IndexError& e) {
        PyErr_SetString(PyExc_IndexError, e.what_without_backtrace());
    } catch (const c10::Error& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

#define SHIFTATTN_CALL(name) PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n)

// the allocator of workspaces, then the addresses of `names`
SHIFTATTN_CALL(bind) {
    if (n != 1 + kFunctions) {
        PyErr_Format(PyExc_TypeError, "an allocator and %zd addresses wanted, not %zd arguments", kFunctions, n);
        return nullptr;
    }
    void* at[kFunctions];
    for (Py_ssize_t i = 0; i < kFunctions; ++i) {
        at[i] = PyLong_AsVoidPtr(a[1 + i]);
        if (!at[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function of the library has no address");
            return nullptr;
        }
    }
    memcpy(&lib, at, sizeof(lib));
    Py_INCREF(a[0]);
    Py_XSETREF(allocate, a[0]);
    Py_RETURN_NONE;
}

// qkv, send, P, h, h_kv
SHIFTATTN_CALL(pack_seq2head) {
    return run(n, 5, [&] {
        const at::Tensor &qkv = tensor(a[0]), &send = tensor(a[1]);
        const int32_t P = whole(a[2]), h = whole(a[3]), h_kv = whole(a[4]);
        dims(qkv, 3, "qkv");
        dims(send, 4, "send");
        need(qkv.size(1) == h + 2 * static_cast<int64_t>(h_kv) && qkv.is_contiguous() && send.is_contiguous() && send.scalar_type() == qkv.scalar_type() &&
                 send.size(0) == P && send.size(3) == qkv.size(2),
             "qkv: contiguous [T, h + 2 h_kv, D], send: contiguous [P, T_pad, .., D] of its type");
        // (heads that P ranks cannot share are the library's to refuse)
        if (P > 0 && h % P == 0 && h_kv >= 0 && (h_kv % P == 0 || P % h_kv == 0))
            need(send.size(2) == h / P + 2 * local_kv_heads(P, h_kv), "send: [P, T_pad, hq_l + 2 hkv_l, D]");
        return [x = exchange(P, h, h_kv, qkv.size(2), dtype_code(qkv)), in = ptr(qkv), out = ptr(send), T = cut(qkv.size(0)), T_pad = cut(send.size(1)),
                st = stream()] { return lib.pack(in, out, T, T_pad, &x, st); };
    });
}

// recv, out
SHIFTATTN_CALL(unpack_head2seq) {
    return run(n, 2, [&] {
        const at::Tensor &recv = tensor(a[0]), &out = tensor(a[1]);
        dims(recv, 4, "recv");
        dims(out, 3, "out");
        const int64_t P = recv.size(0), h = out.size(1);
        need(out.size(2) == recv.size(3) && h == P * recv.size(2) && recv.is_contiguous() && out.is_contiguous() && out.scalar_type() == recv.scalar_type(),
             "recv: contiguous [P, T_pad, h / P, D], out: contiguous [T, h, D] of its type");
        return [x = exchange(P, h, 0, recv.size(3), dtype_code(recv)), in = ptr(recv), to = ptr(out), T = cut(out.size(0)), T_pad = cut(recv.size(1)),
                st = stream()] { return lib.unpack(in, to, T, T_pad, &x, st); };
    });
}

// q, kv_cache, block_table, cu_seqlens_q, seq_lens, max_q_len, max_seq_len, out, softmax_scale, k_new, v_new, slot_mapping, workspace,
// k_scale, v_scale
SHIFTATTN_CALL(prefill) {
    Owned own;
    return run(n, 15, [&] {
        const at::Tensor &q = tensor(a[0]), &cache = tensor(a[1]), &table = tensor(a[2]), &cu = tensor(a[3]), &lens = tensor(a[4]), &out = tensor(a[7]);
        const at::Tensor *k = tensor_or_none(a[9]), *v = tensor_or_none(a[10]), *slots = tensor_or_none(a[11]);
        const int64_t seqs = lens.size(0);
        need(cu.scalar_type() == at::kInt && lens.scalar_type() == at::kInt && cu.size(0) == seqs + 1 && cu.is_contiguous() && lens.is_contiguous(),
             "cu_seqlens_q, seq_lens: contiguous int32 [num_seqs + 1], [num_seqs]");
        need(out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type(), "out: shape and type of q");
        const shiftattn_attn d = describe(q, cache, table, a[8], k, &out, a[13], a[14]);
        need(table.size(0) >= seqs, "block_table: a row per sequence");
        rows_of(q, out, k, v, slots, cache);
        const int32_t mq = whole(a[5]), ms = whole(a[6]);
        const at::Tensor* ws = workspace(a[12], a[0], own, [&] { return lib.prefill_bytes(cut(seqs), cut(q.size(0)), mq, ms, &d); });
        return [d, pq = ptr(q), pk = ptr(k), pv = ptr(v), ps = ptr(slots), pc = ptr(cache), pt = ptr(table), pu = ptr(cu), pl = ptr(lens), seqs = cut(seqs),
                rows = cut(q.size(0)), mq, ms, po = ptr(out), pw = ptr(ws), nw = bytes(ws), st = stream()] {
            return lib.prefill(pq, pk, pv, static_cast<int64_t*>(ps), pc, static_cast<int32_t*>(pt), static_cast<int32_t*>(pu), static_cast<int32_t*>(pl),
                               seqs, rows, mq, ms, po, pw, nw, &d, st);
        };
    });
}

// q, kv_cache, block_table, seq_lens, max_seq_len, out, softmax_scale, k_new, v_new, slot_mapping, workspace, k_scale, v_scale; owned: the
// library's scratch memory instead of a workspace
PyObject* decode_call(PyObject* const* a, Py_ssize_t n, bool owned) {
    Owned own;
    return run(n, 13, [&] {
        const at::Tensor &q = tensor(a[0]), &cache = tensor(a[1]), &table = tensor(a[2]), &lens = tensor(a[3]), &out = tensor(a[5]);
        const at::Tensor *k = tensor_or_none(a[7]), *v = tensor_or_none(a[8]), *slots = tensor_or_none(a[9]);
        dims(q, 3, "q");
        need(lens.scalar_type() == at::kInt && lens.size(0) == q.size(0) && lens.is_contiguous(), "seq_lens: contiguous int32 [num_seqs]");
        need(out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type(), "out: shape and type of q");
        const shiftattn_attn d = describe(q, cache, table, a[6], k, &out, a[11], a[12]);
        need(table.size(0) >= q.size(0), "block_table: a row per sequence");
        rows_of(q, out, k, v, slots, cache);
        const int32_t ms = whole(a[4]);
        const at::Tensor* ws = owned ? nullptr : workspace(a[10], a[0], own, [&] { return lib.decode_bytes(cut(q.size(0)), ms, &d); });
        return [d, pq = ptr(q), pk = ptr(k), pv = ptr(v), ps = ptr(slots), pc = ptr(cache), pt = ptr(table), pl = ptr(lens), seqs = cut(q.size(0)), ms,
                po = ptr(out), pw = ptr(ws), nw = bytes(ws), st = stream(), owned] {
            const auto* slot = static_cast<int64_t*>(ps);
            const auto *blocks = static_cast<int32_t*>(pt), *len = static_cast<int32_t*>(pl);
            return owned ? lib.decode_static(pq, pk, pv, slot, pc, blocks, len, seqs, ms, po, &d, st)
                         : lib.decode(pq, pk, pv, slot, pc, blocks, len, seqs, ms, po, pw, nw, &d, st);
        };
    });
}
SHIFTATTN_CALL(decode) { return decode_call(a, n, false); }
SHIFTATTN_CALL(decode_static) { return decode_call(a, n, true); }

// q, kv_cache, block_table, cu_seqlens_q, seq_lens, num_prefill_seqs, max_q_len, max_prefill_seq_len, max_decode_seq_len, out, softmax_scale,
// k_new, v_new, slot_mapping, workspace, k_scale, v_scale
SHIFTATTN_CALL(mixed) {
    Owned own;
    return run(n, 17, [&] {
        const at::Tensor &q = tensor(a[0]), &cache = tensor(a[1]), &table = tensor(a[2]), &cu = tensor(a[3]), &lens = tensor(a[4]), &out = tensor(a[9]);
        const at::Tensor *k = tensor_or_none(a[11]), *v = tensor_or_none(a[12]), *slots = tensor_or_none(a[13]);
        dims(q, 3, "q");
        const int64_t chunks = whole(a[5]), rows = lens.size(0) - chunks, chunk_rows = q.size(0) - rows;
        need(rows >= 0 && chunk_rows >= 0 && cu.size(0) == chunks + 1, "cu_seqlens_q: [num_prefill_seqs + 1], one row of q per other sequence");
        need(cu.scalar_type() == at::kInt && lens.scalar_type() == at::kInt && cu.is_contiguous() && lens.is_contiguous(), "cu_seqlens_q, seq_lens: contiguous int32");
        need(out.sizes() == q.sizes() && out.scalar_type() == q.scalar_type() && table.size(0) == lens.size(0), "out: shape and type of q; block_table: a row per sequence");
        const shiftattn_attn d = describe(q, cache, table, a[10], k, &out, a[15], a[16]);
        rows_of(q, out, k, v, slots, cache);
        const int32_t mq = whole(a[6]), mp = whole(a[7]), md = whole(a[8]);
        const at::Tensor* ws = workspace(a[14], a[0], own, [&] { return lib.mixed_bytes(cut(chunks), cut(chunk_rows), mq, mp, cut(rows), md, &d); });
        return [d, pq = ptr(q), pk = ptr(k), pv = ptr(v), ps = ptr(slots), pc = ptr(cache), pt = ptr(table), pu = ptr(cu), pl = ptr(lens),
                chunks = cut(chunks), chunk_rows = cut(chunk_rows), mq, mp, rows = cut(rows), md, po = ptr(out), pw = ptr(ws), nw = bytes(ws), st = stream()] {
            return lib.mixed(pq, pk, pv, static_cast<int64_t*>(ps), pc, static_cast<int32_t*>(pt), static_cast<int32_t*>(pu), static_cast<int32_t*>(pl),
                             chunks, chunk_rows, mq, mp, rows, md, po, pw, nw, &d, st);
        };
    });
}

// q, kv_cache, block_table, softmax_scale, k_new, out, k_scale, v_scale -> the descriptor's bytes
SHIFTATTN_CALL(attn_desc) {
    PyObject* bytes = nullptr;
    PyObject* done = run(n, 8, [&] {
        const shiftattn_attn d = describe(tensor(a[0]), tensor(a[1]), tensor(a[2]), a[3], tensor_or_none(a[4]), tensor_or_none(a[5]), a[6], a[7]);
        bytes = PyBytes_FromStringAndSize(reinterpret_cast<const char*>(&d), sizeof(d));
        if (!bytes) throw PythonError{};
        return [] { return 0; };
    });
    Py_XDECREF(done);
    return bytes;
}

// k_new, v_new, slot_mapping, kv_cache, k_scale, v_scale
SHIFTATTN_CALL(kv_write) {
    return run(n, 6, [&] {
        const at::Tensor &k = tensor(a[0]), &v = tensor(a[1]), &slots = tensor(a[2]), &cache = tensor(a[3]);
        dims(k, 3, "k_new");
        apart(k);
        need(v.sizes() == k.sizes() && v.scalar_type() == k.scalar_type() && slots.scalar_type() == at::kLong && slots.size(0) == k.size(0) &&
                 slots.is_contiguous() && row_stride(v) == row_stride(k),
             "v_new: shape, type and row stride of k_new; slot_mapping: contiguous int64 [n_tokens]");
        dims(cache, 4, "kv_cache");
        need(cache.size(1) == k.size(1) && cache.size(2) == 2 && cache.size(3) == kBlock * k.size(2) && cache.is_contiguous() &&
                 (cache.scalar_type() == at::kByte || cache.scalar_type() == k.scalar_type()),
             "kv_cache: contiguous [num_blocks, hkv_l, 2, 16 * D] of k_new's type or uint8");
        shiftattn_attn d{};
        d.num_q_heads = d.num_kv_heads = cut(k.size(1)), d.head_dim = cut(k.size(2)), d.dtype = dtype_code(k), d.block_size = kBlock;
        d.num_blocks = cut(cache.size(0)), d.softmax_scale = 1.0f, d.kv_stride = row_stride(k);
        d.kv_format = cache.scalar_type() == at::kByte ? SHIFTATTN_KV_FP8_E4M3 : SHIFTATTN_KV_SAME;
        d.k_scale = real(a[4]), d.v_scale = real(a[5]);
        return [d, pk = ptr(k), pv = ptr(v), ps = ptr(slots), rows = cut(k.size(0)), pc = ptr(cache), st = stream()] {
            return lib.kv_write(pk, pv, static_cast<int64_t*>(ps), rows, pc, &d, st);
        };
    });
}

// x, w_qkv, send, P, h, h_kv, workspace
SHIFTATTN_CALL(qkv_proj_pack) {
    return run(n, 7, [&] {
        const at::Tensor &x = tensor(a[0]), &w = tensor(a[1]), &send = tensor(a[2]);
        const at::Tensor* ws = dense_or_none(a[6]);
        const int64_t P = whole(a[3]), h = whole(a[4]), h_kv = whole(a[5]);
        dims(x, 2, "x");
        dims(w, 2, "w_qkv");
        dims(send, 4, "send");
        const int64_t D = send.size(3);
        need(w.size(0) == (h + 2 * h_kv) * D && w.size(1) == x.size(1) && x.is_contiguous() && w.is_contiguous() && send.is_contiguous(),
             "x [T, d_model], w_qkv [(h + 2 h_kv) D, d_model], send: contiguous");
        need(P > 0 && send.size(0) == P && send.size(2) == h / P + 2 * local_kv_heads(P, h_kv) && x.scalar_type() == w.scalar_type() &&
                 w.scalar_type() == send.scalar_type(),
             "send: [P, T_pad, hq_l + 2 hkv_l, D], one type");
        return [xc = exchange(P, h, h_kv, D, dtype_code(x)), px = ptr(x), pw = ptr(w), po = ptr(send), T = cut(x.size(0)), T_pad = cut(send.size(1)),
                d = cut(x.size(1)), given = ws != nullptr, pk = ptr(ws), nk = bytes(ws), st = stream()] {
            return given ? lib.qkv(px, pw, po, T, T_pad, d, &xc, pk, nk, st) : lib.qkv_plain(px, pw, po, T, T_pad, d, &xc, st);
        };
    });
}

// recv, w_o, out, workspace
SHIFTATTN_CALL(unpack_o_proj) {
    return run(n, 4, [&] {
        const at::Tensor &recv = tensor(a[0]), &w = tensor(a[1]), &out = tensor(a[2]);
        const at::Tensor* ws = dense_or_none(a[3]);
        dims(recv, 4, "recv");
        dims(w, 2, "w_o");
        dims(out, 2, "out");
        const int64_t P = recv.size(0), h = P * recv.size(2), D = recv.size(3);
        need(w.size(0) == out.size(1) && w.size(1) == h * D && recv.is_contiguous() && w.is_contiguous() && out.is_contiguous() &&
                 recv.scalar_type() == w.scalar_type() && w.scalar_type() == out.scalar_type(),
             "recv [P, T_pad, hq_l, D], w_o [d_model, h D], out [T, d_model]: contiguous, one type");
        return [xc = exchange(P, h, 0, D, dtype_code(recv)), pr = ptr(recv), pw = ptr(w), po = ptr(out), T = cut(out.size(0)), T_pad = cut(recv.size(1)),
                d = cut(out.size(1)), given = ws != nullptr, pk = ptr(ws), nk = bytes(ws), st = stream()] {
            return given ? lib.o_proj(pr, pw, po, T, T_pad, d, &xc, pk, nk, st) : lib.o_proj_plain(pr, pw, po, T, T_pad, d, &xc, st);
        };
    });
}

// x, codes, scales
SHIFTATTN_CALL(quantize_rows_fp8) {
    return run(n, 3, [&] {
        const at::Tensor &x = tensor(a[0]), &codes = tensor(a[1]), &scales = tensor(a[2]);
        dims(x, 2, "x");
        need(x.scalar_type() == at::kBFloat16 && codes.scalar_type() == at::kByte && scales.scalar_type() == at::kFloat, "x bfloat16, codes uint8, scales float32");
        need(codes.sizes() == x.sizes() && scales.dim() == 1 && scales.size(0) == x.size(0) && x.is_contiguous() && codes.is_contiguous() && scales.is_contiguous(),
             "codes: shape of x, scales: [rows], contiguous");
        return [px = ptr(x), pc = ptr(codes), ps = ptr(scales), rows = cut(x.size(0)), cols = cut(x.size(1)), st = stream()] {
            return lib.quantize_rows(px, pc, static_cast<float*>(ps), rows, cols, st);
        };
    });
}

// recv, codes, scales
SHIFTATTN_CALL(quantize_recv_fp8) {
    return run(n, 3, [&] {
        const at::Tensor &recv = tensor(a[0]), &codes = tensor(a[1]), &scales = tensor(a[2]);
        dims(recv, 4, "recv");
        need(recv.scalar_type() == at::kBFloat16 && codes.scalar_type() == at::kByte && scales.scalar_type() == at::kFloat && codes.sizes() == recv.sizes(),
             "recv bfloat16, codes uint8 of its shape, scales float32");
        need(recv.is_contiguous() && codes.is_contiguous() && scales.is_contiguous(), "recv, codes, scales: contiguous");
        return [x = exchange(recv.size(0), recv.size(0) * recv.size(2), 0, recv.size(3), SHIFTATTN_BF16), pr = ptr(recv), pc = ptr(codes), ps = ptr(scales),
                T = cut(scales.size(0)), T_pad = cut(recv.size(1)), st = stream()] {
            return lib.quantize_recv(pr, pc, static_cast<float*>(ps), T, T_pad, &x, st);
        };
    });
}

// x_codes, x_scales, w_codes, w_scales, send, P, h, h_kv, workspace
SHIFTATTN_CALL(qkv_proj_pack_fp8) {
    return run(n, 9, [&] {
        const at::Tensor &x = tensor(a[0]), &xs = tensor(a[1]), &w = tensor(a[2]), &ws = tensor(a[3]), &send = tensor(a[4]);
        const at::Tensor* work = dense_or_none(a[8]);
        const int64_t P = whole(a[5]), h = whole(a[6]), h_kv = whole(a[7]);
        dims(x, 2, "x_codes");
        dims(w, 2, "w_codes");
        dims(send, 4, "send");
        const int64_t D = send.size(3);
        need(x.scalar_type() == at::kByte && w.scalar_type() == at::kByte && xs.scalar_type() == at::kFloat && ws.scalar_type() == at::kFloat &&
                 send.scalar_type() == at::kBFloat16,
             "codes uint8, scales float32, send bfloat16");
        need(w.size(0) == (h + 2 * h_kv) * D && w.size(1) == x.size(1) && xs.dim() == 1 && xs.size(0) == x.size(0) && ws.dim() == 1 && ws.size(0) == w.size(0) &&
                 P > 0 && send.size(0) == P && send.size(2) == h / P + 2 * local_kv_heads(P, h_kv),
             "x [T, d_model], w [(h + 2 h_kv) D, d_model], a scale per row, send [P, T_pad, hq_l + 2 hkv_l, D]");
        need(x.is_contiguous() && xs.is_contiguous() && w.is_contiguous() && ws.is_contiguous() && send.is_contiguous(), "contiguous");
        return [xc = exchange(P, h, h_kv, D, SHIFTATTN_BF16), px = ptr(x), pxs = ptr(xs), pw = ptr(w), pws = ptr(ws), po = ptr(send), T = cut(x.size(0)),
                T_pad = cut(send.size(1)), d = cut(x.size(1)), pk = ptr(work), nk = bytes(work), st = stream()] {
            return lib.qkv_fp8(px, static_cast<float*>(pxs), pw, static_cast<float*>(pws), po, T, T_pad, d, &xc, pk, nk, st);
        };
    });
}

// recv_codes, a_scales, w_codes, w_scales, out, workspace
SHIFTATTN_CALL(unpack_o_proj_fp8) {
    return run(n, 6, [&] {
        const at::Tensor &recv = tensor(a[0]), &as = tensor(a[1]), &w = tensor(a[2]), &ws = tensor(a[3]), &out = tensor(a[4]);
        const at::Tensor* work = dense_or_none(a[5]);
        dims(recv, 4, "recv_codes");
        dims(w, 2, "w_codes");
        dims(out, 2, "out");
        const int64_t P = recv.size(0), h = P * recv.size(2), D = recv.size(3);
        need(recv.scalar_type() == at::kByte && w.scalar_type() == at::kByte && as.scalar_type() == at::kFloat && ws.scalar_type() == at::kFloat &&
                 out.scalar_type() == at::kBFloat16,
             "codes uint8, scales float32, out bfloat16");
        need(w.size(0) == out.size(1) && w.size(1) == h * D && as.size(0) >= out.size(0) && ws.dim() == 1 && ws.size(0) == out.size(1),
             "recv [P, T_pad, hq_l, D], w [d_model, h D], a scale per token and per feature, out [T, d_model]");
        need(recv.is_contiguous() && as.is_contiguous() && w.is_contiguous() && ws.is_contiguous() && out.is_contiguous(), "contiguous");
        return [xc = exchange(P, h, 0, D, SHIFTATTN_BF16), pr = ptr(recv), pas = ptr(as), pw = ptr(w), pws = ptr(ws), po = ptr(out), T = cut(out.size(0)),
                T_pad = cut(recv.size(1)), d = cut(out.size(1)), pk = ptr(work), nk = bytes(work), st = stream()] {
            return lib.o_proj_fp8(pr, static_cast<float*>(pas), pw, static_cast<float*>(pws), po, T, T_pad, d, &xc, pk, nk, st);
        };
    });
}

#define SHIFTATTN_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SHIFTATTN_METHOD(bind), SHIFTATTN_METHOD(pack_seq2head), SHIFTATTN_METHOD(unpack_head2seq), SHIFTATTN_METHOD(prefill),
                         SHIFTATTN_METHOD(decode), SHIFTATTN_METHOD(decode_static), SHIFTATTN_METHOD(mixed), SHIFTATTN_METHOD(kv_write),
                         SHIFTATTN_METHOD(qkv_proj_pack), SHIFTATTN_METHOD(unpack_o_proj), SHIFTATTN_METHOD(quantize_rows_fp8),
                         SHIFTATTN_METHOD(quantize_recv_fp8), SHIFTATTN_METHOD(qkv_proj_pack_fp8), SHIFTATTN_METHOD(unpack_o_proj_fp8),
                         SHIFTATTN_METHOD(attn_desc),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    PyObject* m = PyModule_Create(&module);
    PyObject* names = PyTuple_New(kFunctions);
    if (m && names) {
        bool ok = true;
        for (Py_ssize_t i = 0; i < kFunctions; ++i) {
            PyObject* name = PyUnicode_FromString(kNames[i]);
            ok = ok && name;
            PyTuple_SET_ITEM(names, i, name);
        }
        if (ok && PyModule_AddObject(m, "names", names) == 0) return m;   // (takes the reference)
    }
    Py_XDECREF(names);
    Py_XDECREF(m);
    return nullptr;
}
