// The Python side of libactq's device calls in native code: arguments from torch tensors, outputs, the current
// stream, errors as Python exceptions, and the autograd functions of the layers whose arithmetic is short.
//
// A small call is bound by the host.  With ctypes and the checks in Python it took 5.2 to 5.9 us, of which the
// launch is 2.4; here it takes 2.9 to 3.9 (compression and decompression of [4, 4096], five calls: 32.7 -> 19.3 us
// from one to the next).  A layer's autograd function in Python costs
// more than its kernels: its backward half takes the interpreter's lock on the autograd thread, behind the
// thread that waits for it.
//
// libactq itself knows nothing of torch: its entry points arrive as addresses (attach), so that this file and
// the library are built and replaced independently.
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <initializer_list>
#include <optional>
#include <string>
#include <vector>

#include <torch/extension.h>

#include <ATen/TensorSubclassLikeUtils.h>
#include <ATen/autocast_mode.h>
#include <c10/core/GradMode.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include "actq.h"

namespace {

using at::Tensor;

struct Api {
    decltype(&actq_last_error) last_error;
    decltype(&actq_group_stats) group_stats;
    decltype(&actq_sample_sensitivity) sample_sensitivity;
    decltype(&actq_allocate_bits_device) allocate_bits_device;
    decltype(&actq_quantize_pack) quantize_pack;
    decltype(&actq_unpack_dequantize) unpack_dequantize;
    decltype(&actq_relu_mask_bytes) relu_mask_bytes;
    decltype(&actq_relu_forward) relu_forward;
    decltype(&actq_relu_backward) relu_backward;
    decltype(&actq_pool2d_output_size) pool2d_output_size;
    decltype(&actq_maxpool2d_forward) maxpool2d_forward;
    decltype(&actq_maxpool2d_backward) maxpool2d_backward;
    decltype(&actq_linear_backward) linear_backward;
};
Api api = {};
PyObject* actq_error = nullptr;   // the binding's exception class, called with (code, message)

constexpr int32_t kG = 256;

// ----------------------------------------------------------------------------- errors and arguments

// Python exceptions are raised from threads with and without the interpreter's lock (the autograd functions run without
// it, their backward halves on threads of their own): both of these take it, and the error travels in the C++ exception.
[[noreturn]] void throw_pending()   // under the lock
{
    python_error error;
    error.persist();
    throw error;
}

[[noreturn]] void raise(int code)
{
    const std::string message = api.last_error();   // of this thread
    pybind11::gil_scoped_acquire gil;
    PyObject* e = PyObject_CallFunction(actq_error, "is", code, message.c_str());
    if (e) {
        PyErr_SetObject(actq_error, e);
        Py_DECREF(e);
    }
    throw_pending();
}

[[noreturn]] void python_exception(PyObject* type, const char* message)
{
    pybind11::gil_scoped_acquire gil;
    PyErr_SetString(type, message);
    throw_pending();
}

// A call of the library; its status becomes the binding's exception.  The interpreter's lock is released
// for the call if this thread holds it.
template <typename... Params, typename... Args>
void call(int (*f)(Params...), Args... args)
{
    int code;
    if (PyGILState_Check()) {
        pybind11::gil_scoped_release no_gil;
        code = f(args...);
    } else {
        code = f(args...);
    }
    if (code != ACTQ_OK) raise(code);
}

const Tensor& tensor_of(PyObject* o, const char* name)
{
    TORCH_CHECK_TYPE(THPVariable_Check(o), name, " must be a torch tensor");
    return THPVariable_Unpack(o);
}

std::optional<Tensor> optional_tensor(PyObject* o, const char* name)
{
    if (o == Py_None) return std::nullopt;
    return tensor_of(o, name);
}

std::string dtype_name(at::ScalarType type)
{
    return type == at::kFloat ? "torch.float32" : type == at::kHalf ? "torch.float16" : type == at::kByte ? "torch.uint8"
         : type == at::kLong ? "torch.int64" : type == at::kShort ? "torch.int16" : type == at::kDouble ? "torch.float64"
         : type == at::kBFloat16 ? "torch.bfloat16" : std::string(c10::toString(type));
}

// A tensor's memory, checked, as whatever pointer the callee takes.  A function's arguments are evaluated in any order:
// the pointers of a call are made one by one in front of it, so that the first wrong argument is the one reported, and
// before the stream is asked for.
struct Memory {
    void* p;
    template <typename T>
    operator T*() const { return static_cast<T*>(p); }
};

Memory on_gpu(const Tensor& t, const char* name)
{
    TORCH_CHECK_VALUE(t.is_cuda(), name, " must live on the GPU");
    TORCH_CHECK_VALUE(t.is_contiguous(), name, " must be contiguous");
    return {t.data_ptr()};
}

Memory on_gpu(const Tensor& t, at::ScalarType type, const char* name)
{
    const Memory m = on_gpu(t, name);
    TORCH_CHECK_TYPE(t.scalar_type() == type, name, " must be ", dtype_name(type), ", got ", dtype_name(t.scalar_type()));
    return m;
}

actq_dtype dtype_of(const Tensor& t)
{
    if (t.scalar_type() == at::kFloat) return ACTQ_F32;
    TORCH_CHECK_TYPE(t.scalar_type() == at::kHalf, "unsupported dtype ", dtype_name(t.scalar_type()));
    return ACTQ_F16;
}

// A tensor as [N, D].
struct View {
    int64_t N, D, groups;   // groups of a sample
};

// The size of a group, as the sizes of the outputs are worked out with it and as the library is told: one number.
int32_t group_size(int64_t G)
{
    if (G == 0) python_exception(PyExc_ZeroDivisionError, "G must not be 0");
    TORCH_CHECK_VALUE(G > 0 && G <= INT32_MAX, "G must be positive and fit 32 bits, got ", G);
    return static_cast<int32_t>(G);
}

View view_of(const Tensor& x, int32_t G = kG)
{
    if (x.dim() == 0) python_exception(PyExc_IndexError, "a tensor without dimensions has no samples");
    if (x.size(0) == 0) python_exception(PyExc_ZeroDivisionError, "no samples");
    View v;
    v.N = x.size(0);
    v.D = x.numel() / v.N;
    v.groups = (v.D + G - 1) / G;
    return v;
}

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// The handle of a torch stream, or of the current device's current stream.
void* stream_of(PyObject* o)
{
    if (o == Py_None) return current_stream();
    PyObject* handle = PyObject_GetAttrString(o, "cuda_stream");
    if (!handle) throw python_error();
    void* s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (PyErr_Occurred()) throw python_error();
    return s;
}

int64_t integer(PyObject* o)
{
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw python_error();
    return v;
}

// The lower 64 bits of a Python integer.
uint64_t word(PyObject* o)
{
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == static_cast<unsigned long long>(-1) && PyErr_Occurred()) throw python_error();
    return v;
}

Tensor empty_on(const Tensor& like, at::IntArrayRef shape, at::ScalarType type)
{
    return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

PyObject* give(PyObject* passed, const Tensor& made)
{
    if (passed == Py_None) return THPVariable_Wrap(made);
    Py_INCREF(passed);
    return passed;
}

PyObject* tuple_of(std::initializer_list<PyObject*> items)
{
    PyObject* t = PyTuple_New(static_cast<Py_ssize_t>(items.size()));
    Py_ssize_t k = 0;
    for (PyObject* o : items) {
        if (!t || !o) throw python_error();
        PyTuple_SET_ITEM(t, k++, o);
    }
    return t;
}

// Every entry takes its arguments by position (the binding names them) and in full.
#define ACTQ_ENTRY(NAME, COUNT)                                                                                   \
    PyObject* NAME(PyObject*, PyObject* const* a, Py_ssize_t n)                                                   \
    {                                                                                                             \
        HANDLE_TH_ERRORS                                                                                          \
        TORCH_CHECK_TYPE(n == COUNT, #NAME " takes " #COUNT " arguments");                                        \
        return NAME##_impl(a);                                                                                    \
        END_HANDLE_TH_ERRORS                                                                                      \
    }

// ----------------------------------------------------------------------------- the codec

// (x, gmin or None, grange or None, G, stream or None) -> (gmin, grange)
PyObject* group_stats_impl(PyObject* const* a)
{
    const Tensor& x = tensor_of(a[0], "x");
    const int32_t G = group_size(integer(a[3]));
    TORCH_CHECK_VALUE(x.is_cuda(), "x must live on the GPU");
    const View v = view_of(x, G);
    const Tensor gmin = a[1] == Py_None ? empty_on(x, {v.N, v.groups}, at::kFloat) : tensor_of(a[1], "gmin");
    const Tensor grange = a[2] == Py_None ? empty_on(x, {v.N, v.groups}, at::kFloat) : tensor_of(a[2], "grange");
    TORCH_CHECK_VALUE(gmin.numel() == v.N * v.groups && grange.numel() == v.N * v.groups, "gmin / grange must hold N*ng floats");
    const Memory xp = on_gpu(x, "x");
    const actq_dtype dt = dtype_of(x);
    const Memory lo = on_gpu(gmin, at::kFloat, "gmin"), range = on_gpu(grange, at::kFloat, "grange");
    call(api.group_stats, xp, dt, v.N, v.D, G, lo, range, stream_of(a[4]));
    return tuple_of({give(a[1], gmin), give(a[2], grange)});
}
ACTQ_ENTRY(group_stats, 5)

// (grange, grad2 or None, w or None, G, stream or None) -> w
PyObject* sample_sensitivity_impl(PyObject* const* a)
{
    const Tensor& grange = tensor_of(a[0], "grange");
    TORCH_CHECK_VALUE(grange.dim() == 2, "grange must be [N, ng]");
    const int64_t N = grange.size(0), ng = grange.size(1);
    TORCH_CHECK_VALUE(grange.is_cuda(), "grange must live on the GPU");
    const std::optional<Tensor> grad2 = optional_tensor(a[1], "grad2");
    const Tensor w = a[2] == Py_None ? empty_on(grange, {N}, at::kFloat) : tensor_of(a[2], "w");
    TORCH_CHECK_VALUE(w.numel() == N && (!grad2 || grad2->numel() == N), "w and grad2 must have N entries");
    const Memory g2 = grad2 ? on_gpu(*grad2, at::kFloat, "grad2") : Memory{nullptr};
    const Memory range = on_gpu(grange, at::kFloat, "grange"), wp = on_gpu(w, at::kFloat, "w");
    call(api.sample_sensitivity, range, N, ng, static_cast<int32_t>(integer(a[3])), g2, wp, stream_of(a[4]));
    return give(a[2], w);
}
ACTQ_ENTRY(sample_sensitivity, 5)

// (w, D: int or tensor, budget, widths, bits or None, offsets or None, result or None, G, stream or None)
// -> (bits, offsets, result)
PyObject* allocate_bits_device_impl(PyObject* const* a)
{
    const Tensor& w = tensor_of(a[0], "w");
    const int64_t M = w.numel();
    TORCH_CHECK_VALUE(w.is_cuda(), "w must live on the GPU");
    const Tensor bits = a[4] == Py_None ? empty_on(w, {M}, at::kByte) : tensor_of(a[4], "bits");
    const Tensor offsets = a[5] == Py_None ? empty_on(w, {M}, at::kLong) : tensor_of(a[5], "offsets");
    const Tensor result = a[6] == Py_None ? empty_on(w, {2}, at::kLong) : tensor_of(a[6], "result");
    TORCH_CHECK_VALUE(bits.numel() == M && offsets.numel() == M && result.numel() == 2, "bits and offsets must have M entries, result 2");
    Memory items = {nullptr};
    int64_t uniform = 0;
    if (PyLong_Check(a[1])) {
        uniform = static_cast<int64_t>(word(a[1]));
    } else {
        const Tensor& D = tensor_of(a[1], "D");
        TORCH_CHECK_VALUE(D.numel() == M, "D must have M entries");
        items = on_gpu(D, at::kLong, "D");
    }
    const Memory wp = on_gpu(w, at::kFloat, "w"), bp = on_gpu(bits, at::kByte, "bits"), op = on_gpu(offsets, at::kLong, "offsets");
    const Memory rp = on_gpu(result, at::kLong, "result");
    call(api.allocate_bits_device, wp, items, uniform, M, static_cast<int32_t>(integer(a[7])), static_cast<int64_t>(word(a[2])),
         static_cast<uint32_t>(word(a[3])), bp, op, rp, stream_of(a[8]));
    return tuple_of({give(a[4], bits), give(a[5], offsets), give(a[6], result)});
}
ACTQ_ENTRY(allocate_bits_device, 9)

Memory header_pointer(const Tensor& header, int64_t groups, int64_t hf)
{
    const at::ScalarType want = hf == ACTQ_HDR_BF16 ? at::kShort : at::kFloat;
    TORCH_CHECK_TYPE(header.scalar_type() == want, "header must be ", dtype_name(want), " for this header format, got ", dtype_name(header.scalar_type()));
    TORCH_CHECK_VALUE(header.numel() == (hf == ACTQ_HDR_TENSOR ? 2 : groups * 2), "header must hold N*ng*2 entries (2 for ACTQ_HDR_TENSOR)");
    return on_gpu(header, want, "header");
}

// (x, bits, offsets, packed, header, seed, tag, noise_bits, G, stream or None, hf)
PyObject* quantize_pack_impl(PyObject* const* a)
{
    const Tensor &x = tensor_of(a[0], "x"), &bits = tensor_of(a[1], "bits"), &offsets = tensor_of(a[2], "offsets");
    const Tensor &packed = tensor_of(a[3], "packed"), &header = tensor_of(a[4], "header");
    const int32_t G = group_size(integer(a[8]));
    const int64_t hf = integer(a[10]);
    const View v = view_of(x, G);
    TORCH_CHECK_VALUE(bits.numel() == v.N && offsets.numel() == v.N, "bits and offsets must have N entries");
    const Memory xp = on_gpu(x, "x");
    const actq_dtype dt = dtype_of(x);
    const Memory bp = on_gpu(bits, at::kByte, "bits"), op = on_gpu(offsets, at::kLong, "offsets"), pp = on_gpu(packed, at::kByte, "packed");
    const Memory hp = header_pointer(header, v.N * v.groups, hf);
    call(api.quantize_pack, xp, dt, v.N, v.D, G, bp, op, word(a[5]), word(a[6]), static_cast<int32_t>(integer(a[7])), pp,
         static_cast<uint64_t>(packed.numel()), hp, static_cast<actq_header_format>(hf), stream_of(a[9]));
    return tuple_of({give(a[3], packed), give(a[4], header)});
}
ACTQ_ENTRY(quantize_pack, 11)

// The second halves (decompress, relu_backward_call, maxpool_backward_call) check the sizes of what the first halves left for
// both of their callers: in the autograd functions it comes from the saved tensors, and those from hooks that may return any tensor.
// `stream`: None or a torch stream; null without the interpreter's lock, for the current one.
void decompress(const Tensor& packed, const Tensor& header, const Tensor& bits, const Tensor& offsets, const Tensor& out, const View& v, int32_t G,
                int64_t hf, PyObject* stream)
{
    TORCH_CHECK_VALUE(bits.numel() == v.N && offsets.numel() == v.N, "bits and offsets must have N entries");
    const Memory pp = on_gpu(packed, at::kByte, "packed"), hp = header_pointer(header, v.N * v.groups, hf);
    const Memory bp = on_gpu(bits, at::kByte, "bits"), op = on_gpu(offsets, at::kLong, "offsets"), xp = on_gpu(out, "out");
    const actq_dtype dt = dtype_of(out);
    call(api.unpack_dequantize, pp, static_cast<uint64_t>(packed.numel()), hp, static_cast<actq_header_format>(hf), bp, op, v.N, v.D, G, xp, dt,
         stream ? stream_of(stream) : current_stream());
}

// (packed, header, bits, offsets, out, G, stream or None, hf) -> out
PyObject* unpack_dequantize_impl(PyObject* const* a)
{
    const Tensor &packed = tensor_of(a[0], "packed"), &header = tensor_of(a[1], "header"), &bits = tensor_of(a[2], "bits");
    const Tensor &offsets = tensor_of(a[3], "offsets"), &out = tensor_of(a[4], "out");
    const int32_t G = group_size(integer(a[5]));
    const int64_t hf = integer(a[7]);
    decompress(packed, header, bits, offsets, out, view_of(out, G), G, hf, a[6]);
    return give(a[4], out);
}
ACTQ_ENTRY(unpack_dequantize, 8)

// How an activation is compressed: mixed widths under a budget, or given ones.
struct Config {
    int64_t budget = 0, capacity = 0;   // bits; bytes of the stream
    uint32_t widths = 0;
    uint64_t seed = 0, tag = 0;
    int32_t noise_bits = 16;
    int64_t hf = ACTQ_HDR_F32;
    std::optional<Tensor> bits, offsets;
};

struct Compressed {
    Tensor bits, offsets, packed, header;
};

// The forward pass of one activation on the current stream: statistics, sensitivities, bit allocation, quantize + pack.
Compressed compress_activation(const Tensor& x, const std::optional<Tensor>& grad2, const Config& c)
{
    const View v = view_of(x);
    const int64_t groups = v.N * v.groups;
    const Memory xp = on_gpu(x, "x");
    const actq_dtype dt = dtype_of(x);
    void* const stream = current_stream();
    Compressed r;
    r.packed = empty_on(x, {c.capacity}, at::kByte);
    r.header = empty_on(x, {groups * 2}, c.hf == ACTQ_HDR_BF16 ? at::kShort : at::kFloat);
    Tensor scratch;   // released when the last call that uses it has been issued, in the order of the stream
    if (c.bits) {
        TORCH_CHECK_VALUE(c.offsets && c.bits->numel() == v.N && c.offsets->numel() == v.N, "bits and offsets must have N entries");
        r.bits = *c.bits;
        r.offsets = *c.offsets;
    } else {
        TORCH_CHECK_VALUE(!grad2 || grad2->numel() == v.N, "grad2 must have N entries");
        const Memory g2 = grad2 ? on_gpu(*grad2, at::kFloat, "grad2") : Memory{nullptr};
        // the allocator's result; then minima, ranges, sensitivities
        scratch = empty_on(x, {2 + (2 * groups + v.N + 1) / 2}, at::kLong);
        r.bits = empty_on(x, {v.N}, at::kByte);
        r.offsets = empty_on(x, {v.N}, at::kLong);
        int64_t* const result = static_cast<int64_t*>(scratch.data_ptr());
        float* const gmin = reinterpret_cast<float*>(result + 2);
        float* const grange = gmin + groups;
        float* const w = grange + groups;
        const Memory bp = {r.bits.data_ptr()}, op = {r.offsets.data_ptr()};
        call(api.group_stats, xp, dt, v.N, v.D, kG, gmin, grange, stream);
        call(api.sample_sensitivity, grange, v.N, v.groups, kG, g2, w, stream);
        call(api.allocate_bits_device, w, nullptr, v.D, v.N, kG, c.budget, c.widths, bp, op, result, stream);
    }
    const Memory bp = on_gpu(r.bits, at::kByte, "bits"), op = on_gpu(r.offsets, at::kLong, "offsets");
    call(api.quantize_pack, xp, dt, v.N, v.D, kG, bp, op, c.seed, c.tag, c.noise_bits, r.packed.data_ptr(), static_cast<uint64_t>(c.capacity),
         r.header.data_ptr(), static_cast<actq_header_format>(c.hf), stream);
    return r;
}

// (budget, widths, capacity, seed, tag, noise_bits, hf, bits or None, offsets or None)
Config config_of(PyObject* const* a)
{
    Config c;
    c.budget = static_cast<int64_t>(word(a[0]));
    c.widths = static_cast<uint32_t>(word(a[1]));
    c.capacity = integer(a[2]);
    c.seed = word(a[3]);
    c.tag = word(a[4]);
    c.noise_bits = static_cast<int32_t>(integer(a[5]));
    c.hf = integer(a[6]);
    c.bits = optional_tensor(a[7], "bits");
    c.offsets = optional_tensor(a[8], "offsets");
    return c;
}

// (x, grad2 or None, budget, widths, capacity, seed, tag, noise_bits, hf) -> (bits, offsets, packed, header)
PyObject* compress_mixed_impl(PyObject* const* a)
{
    const Tensor& x = tensor_of(a[0], "x");
    PyObject* const rest[9] = {a[2], a[3], a[4], a[5], a[6], a[7], a[8], Py_None, Py_None};
    const Compressed c = compress_activation(x, optional_tensor(a[1], "grad2"), config_of(rest));
    return tuple_of({THPVariable_Wrap(c.bits), THPVariable_Wrap(c.offsets), THPVariable_Wrap(c.packed), THPVariable_Wrap(c.header)});
}
ACTQ_ENTRY(compress_mixed, 9)

// ----------------------------------------------------------------------------- exact contexts

int64_t mask_bytes(int64_t n)
{
    uint64_t bytes = 0;
    call(api.relu_mask_bytes, n, &bytes);
    return static_cast<int64_t>(bytes);
}

void relu_forward_call(const Tensor& x, const Tensor& y, const Tensor& mask, PyObject* stream)
{
    const Memory xp = on_gpu(x, "x");
    const actq_dtype dt = dtype_of(x);
    const Memory yp = on_gpu(y, "y"), mp = on_gpu(mask, at::kByte, "mask");
    call(api.relu_forward, xp, dt, x.numel(), yp, mp, stream ? stream_of(stream) : current_stream());
}

void relu_backward_call(const Tensor& mask, const Tensor& grad_y, const Tensor& grad_x, PyObject* stream)
{
    TORCH_CHECK_VALUE(grad_x.numel() == grad_y.numel() && grad_x.scalar_type() == grad_y.scalar_type() && mask.numel() == mask_bytes(grad_y.numel()),
                      "grad_x must match grad_y and mask must have relu_mask_bytes(n) bytes");
    const Memory mp = on_gpu(mask, at::kByte, "mask"), gp = on_gpu(grad_y, "grad_y");
    const actq_dtype dt = dtype_of(grad_y);
    const Memory xp = on_gpu(grad_x, "grad_x");
    call(api.relu_backward, mp, gp, dt, grad_y.numel(), xp, stream ? stream_of(stream) : current_stream());
}

// (x, y or None, mask or None, stream or None) -> (y, mask)
PyObject* relu_forward_impl(PyObject* const* a)
{
    const Tensor& x = tensor_of(a[0], "x");
    const Tensor y = a[1] == Py_None ? at::empty_like(x) : tensor_of(a[1], "y");
    const int64_t bytes = mask_bytes(x.numel());
    const Tensor mask = a[2] == Py_None ? empty_on(x, {bytes}, at::kByte) : tensor_of(a[2], "mask");
    TORCH_CHECK_VALUE(y.numel() == x.numel() && y.scalar_type() == x.scalar_type() && mask.numel() == bytes,
                      "y must match x and mask must have relu_mask_bytes(n) bytes");
    relu_forward_call(x, y, mask, a[3]);
    return tuple_of({give(a[1], y), give(a[2], mask)});
}
ACTQ_ENTRY(relu_forward, 4)

// (mask, grad_y, grad_x or None, stream or None) -> grad_x
PyObject* relu_backward_impl(PyObject* const* a)
{
    const Tensor &mask = tensor_of(a[0], "mask"), &grad_y = tensor_of(a[1], "grad_y");
    const Tensor grad_x = a[2] == Py_None ? at::empty_like(grad_y) : tensor_of(a[2], "grad_x");
    relu_backward_call(mask, grad_y, grad_x, a[3]);
    return give(a[2], grad_x);
}
ACTQ_ENTRY(relu_backward, 4)

// Window of a pooling layer: kernel, stride, padding, dilation, each (rows, columns).
struct Window {
    int32_t k[2], s[2], p[2], d[2];
};

void pair_of(PyObject* o, int32_t (&v)[2])
{
    PyObject* seq = PySequence_Fast(o, "kernel, stride, padding and dilation are pairs");
    if (!seq) throw python_error();
    const bool two = PySequence_Fast_GET_SIZE(seq) == 2;
    long long got[2] = {0, 0};
    if (two)
        for (int i = 0; i < 2; ++i) got[i] = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(seq, i));
    Py_DECREF(seq);
    TORCH_CHECK_TYPE(two, "kernel, stride, padding and dilation are pairs");
    if (PyErr_Occurred()) throw python_error();
    for (int i = 0; i < 2; ++i) v[i] = static_cast<int32_t>(got[i]);
}

Window window_of(PyObject* const* a)
{
    Window w;
    pair_of(a[0], w.k);
    pair_of(a[1], w.s);
    pair_of(a[2], w.p);
    pair_of(a[3], w.d);
    return w;
}

void output_size(int32_t H, int32_t W, const Window& w, int32_t& OH, int32_t& OW)
{
    call(api.pool2d_output_size, H, W, w.k[0], w.k[1], w.s[0], w.s[1], w.p[0], w.p[1], w.d[0], w.d[1], &OH, &OW);
}

// Rows or columns as the library takes them.  Cut to 32 bits, a larger extent would be another image, and the number of planes
// worked out from it would not be that of the outputs.
int32_t extent(int64_t rows_or_columns)
{
    TORCH_CHECK_VALUE(rows_or_columns <= INT32_MAX && rows_or_columns >= INT32_MIN, "rows and columns must fit 32 bits, got ", rows_or_columns);
    return static_cast<int32_t>(rows_or_columns);
}

int32_t extent(const Tensor& t, int64_t dim)
{
    if (t.dim() < 2) python_exception(PyExc_IndexError, "pooling needs rows and columns");
    return extent(t.size(dim));
}

std::vector<int64_t> with_extent(const Tensor& t, int64_t H, int64_t W)
{
    std::vector<int64_t> shape = t.sizes().vec();
    shape[shape.size() - 2] = H;
    shape[shape.size() - 1] = W;
    return shape;
}

// Shapes of a forward call: output extent and planes.
struct Pooling {
    int32_t H, W, OH, OW;
    int64_t planes;
};

Pooling pooling_of(const Tensor& x, const Window& w)
{
    Pooling p;
    p.H = extent(x, -2);
    p.W = extent(x, -1);
    if (p.H == 0 || p.W == 0) python_exception(PyExc_ZeroDivisionError, "no rows or columns");
    p.planes = x.numel() / (static_cast<int64_t>(p.H) * p.W);
    output_size(p.H, p.W, w, p.OH, p.OW);
    return p;
}

void maxpool_forward_call(const Tensor& x, const Pooling& p, const Window& w, const Tensor& y, const Tensor& arg, PyObject* stream)
{
    const Memory xp = on_gpu(x, "x");
    const actq_dtype dt = dtype_of(x);
    const Memory yp = on_gpu(y, "y"), ap = on_gpu(arg, at::kByte, "argmax");
    call(api.maxpool2d_forward, xp, dt, p.planes, p.H, p.W, w.k[0], w.k[1], w.s[0], w.s[1], w.p[0], w.p[1], w.d[0], w.d[1], yp, ap,
         stream ? stream_of(stream) : current_stream());
}

// Shapes of a backward call for images of H x W.
Pooling pooling_of_gradient(const Tensor& grad_y, int32_t H, int32_t W, const Window& w)
{
    Pooling p;
    p.H = H;
    p.W = W;
    output_size(H, W, w, p.OH, p.OW);
    TORCH_CHECK_VALUE(grad_y.dim() >= 2 && grad_y.size(-2) == p.OH && grad_y.size(-1) == p.OW, "grad_y and argmax must be [..., OH, OW]");
    p.planes = grad_y.numel() / (static_cast<int64_t>(p.OH) * p.OW);
    return p;
}

void maxpool_backward_call(const Tensor& arg, const Tensor& grad_y, const Pooling& p, const Window& w, const Tensor& grad_x, PyObject* stream)
{
    TORCH_CHECK_VALUE(arg.numel() == grad_y.numel(), "grad_y and argmax must be [..., OH, OW]");
    TORCH_CHECK_VALUE(grad_x.numel() == p.planes * p.H * p.W && grad_x.scalar_type() == grad_y.scalar_type(), "grad_x must have planes*H*W elements");
    const Memory ap = on_gpu(arg, at::kByte, "argmax"), gp = on_gpu(grad_y, "grad_y");
    const actq_dtype dt = dtype_of(grad_y);
    const Memory xp = on_gpu(grad_x, "grad_x");
    call(api.maxpool2d_backward, ap, gp, dt, p.planes, p.H, p.W, w.k[0], w.k[1], w.s[0], w.s[1], w.p[0], w.p[1], w.d[0], w.d[1], xp,
         stream ? stream_of(stream) : current_stream());
}

// (x, kernel, stride, padding, dilation, y or None, argmax or None, stream or None) -> (y, argmax)
PyObject* maxpool2d_forward_impl(PyObject* const* a)
{
    const Tensor& x = tensor_of(a[0], "x");
    const Window w = window_of(a + 1);
    const Pooling p = pooling_of(x, w);
    const std::vector<int64_t> shape = with_extent(x, p.OH, p.OW);
    const Tensor y = a[5] == Py_None ? empty_on(x, shape, x.scalar_type()) : tensor_of(a[5], "y");
    const Tensor arg = a[6] == Py_None ? empty_on(x, shape, at::kByte) : tensor_of(a[6], "argmax");
    const int64_t outputs = p.planes * p.OH * p.OW;
    TORCH_CHECK_VALUE(y.numel() == outputs && arg.numel() == outputs && y.scalar_type() == x.scalar_type(), "y and argmax must have planes*OH*OW elements");
    maxpool_forward_call(x, p, w, y, arg, a[7]);
    return tuple_of({give(a[5], y), give(a[6], arg)});
}
ACTQ_ENTRY(maxpool2d_forward, 8)

// (argmax, grad_y, H, W, kernel, stride, padding, dilation, grad_x or None, stream or None) -> grad_x
PyObject* maxpool2d_backward_impl(PyObject* const* a)
{
    const Tensor &arg = tensor_of(a[0], "argmax"), &grad_y = tensor_of(a[1], "grad_y");
    const Window w = window_of(a + 4);
    const int32_t H = extent(integer(a[2])), W = extent(integer(a[3]));
    const Pooling p = pooling_of_gradient(grad_y, H, W, w);
    const Tensor grad_x = a[8] == Py_None ? empty_on(grad_y, with_extent(grad_y, p.H, p.W), grad_y.scalar_type()) : tensor_of(a[8], "grad_x");
    maxpool_backward_call(arg, grad_y, p, w, grad_x, a[9]);
    return give(a[8], grad_x);
}
ACTQ_ENTRY(maxpool2d_backward, 10)

// ----------------------------------------------------------------------------- autograd

using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// ----------------------------------------------------------------------------- gradients of a linear layer

struct LinearGradients {
    Tensor x, weight, bias;   // undefined where none was asked for
};

// A tensor whose memory is all there is: no mode, transform or subclass looks on, no tangent of forward-mode differentiation goes with it,
// and nothing is applied lazily.
bool in_memory(const Tensor& t, at::ScalarType type, c10::DeviceIndex device)
{
    return t.defined() && !at::isTensorSubclassLike(t) && t.is_cuda() && t.get_device() == device && t.scalar_type() == type && t.layout() == at::kStrided &&
           t.is_contiguous() && !t.is_neg() && !t._is_zerotensor() && !t._fw_grad(0).defined();
}

// Whether the library's one launch (actq_linear_backward) takes the place of torch's products and sum.  Each product costs the host 18 us
// there and the sum 5, whatever their size; but in a step whose host runs ahead the device's time is what counts, so the launch is for the sizes at
// which it is no slower there.  It loses where a product is few tiles (of 32 x 64) with a long sum, 10 ns per row or output in binary32
// whatever the tiles, and where it is very many tiles, of which each writes little; and, in binary32, to the library's large products.  Products and sum
// of torch -> the launch, device time (us), [rows, inputs, outputs]; in brackets: beyond the rule.
//   binary32  long sums     [128, 1439, 1686] 35 -> 27  ([16, 64, 2048] 15.5 -> 20.8, [16, 576, 1408] 15 -> 17: over the outputs, with few rows)
//                           [1501, 84, 34] 25 -> 17     ([2048, 64, 16] 18.9 -> 21.4, without the input's gradient [1465, 95, 4] 13.8 -> 16.3)
//             many tiles    [171, 40958, 22] 41 -> 31   ([1444, 3613, 7] 30 -> 32, [2048, 4096, 64] 50 -> 53, [1038, 15201, 10] 55 -> 78, [8, 131072, 256] 71 -> 101)
//             products      [128, 2048, 1000] 26 -> 19, [512, 1024, 1000] 37 -> 31  ([512, 2048, 1000] 54 -> 55, [1966, 764, 224] 46 -> 55, [1024, 1024, 1024] 52 -> 57)
//   binary16                [128, 2048, 1000] 27 -> 8, [1024, 1024, 1024] 31 -> 17  ([301, 3881, 1433] 48 -> 52, [8, 21312, 1160] 65 -> 74, [2048, 16384, 10] 51 -> 108)
// Without the sum, which torch makes a kernel of 4 to 8 us, less is gained: binary32 [656, 4992, 16] 15 -> 18, [16, 192, 1464] 12.7 -> 16.3, binary16 [36, 566, 1409]
// 13 -> 15, [1237, 1704, 951] 40 -> 44.  One product alone is torch's: of the input's gradient [128, 2048, 1000] 10.9 -> 15.3, of the weight's [896, 640, 8] 6.4 -> 10.8.
bool one_launch(int64_t rows, int64_t inputs, int64_t outputs, at::ScalarType type, bool need_x, bool need_bias)
{
    if (!need_x && !need_bias) return false;
    if (rows < 1 || rows > 2048 || outputs < ACTQ_LINEAR_MIN_OUTPUTS || outputs > 2048 || inputs < ACTQ_LINEAR_MIN_INPUTS || inputs > ACTQ_LINEAR_MAX_EXTENT) return false;
    // what the library refuses is torch's: a weight of more elements at batch 1, a wide input into two outputs
    if (rows * inputs > ACTQ_LINEAR_MAX_ELEMENTS || outputs * inputs > ACTQ_LINEAR_MAX_ELEMENTS) return false;
    const int64_t columns = (inputs + 63) / 64, tiles_x = (rows + 31) / 32 * columns, tiles_w = (outputs + 31) / 32 * columns, products = rows * inputs * outputs;
    if (type == at::kHalf) {
        if (!need_bias) return outputs <= 1280 && tiles_x <= 2048 && tiles_w <= 2048 && products <= int64_t(1) << 30;
        return tiles_x <= 2560 && tiles_w <= 2560 && products <= int64_t(1) << 31;
    }
    if (!need_bias) return rows <= 768 && outputs <= 768 && tiles_x <= 1024 && tiles_w <= 1024 && products <= int64_t(1) << 27;
    const bool sums = (outputs <= 1280 || rows >= 128) && (rows <= 1024 || outputs >= 32);
    return sums && tiles_x <= (rows <= 512 ? 4096 : 1500) && tiles_w <= 4096 && products < int64_t(1) << (rows <= 768 ? 29 : 28);
}

// The gradients of y = x weight^T + bias by that launch on the current stream; false, and nothing done, where torch's own operators have
// to serve: a graph of the gradients themselves, tangents, autocast, modes and transforms, operands that differ in type or are not plain memory,
// sizes beyond the rule.  `x` is asked for only once all else is settled.
template <typename X>
bool fused_gradients(const Tensor& grad_y, const Tensor& weight, X x_of, at::ScalarType type, int64_t inputs, bool need_x, bool need_weight, bool need_bias,
                     LinearGradients& out)
{
    if (c10::GradMode::is_enabled() || at::autocast::is_autocast_enabled(at::kCUDA) || !need_weight) return false;
    const c10::DeviceIndex device = c10::hip::current_device();
    if ((type != at::kFloat && type != at::kHalf) || !in_memory(grad_y, type, device) || !in_memory(weight, type, device)) return false;
    if (grad_y.dim() < 1 || grad_y.numel() == 0 || weight.dim() != 2 || weight.size(0) != grad_y.size(-1) || weight.size(1) != inputs) return false;
    const int64_t outputs = weight.size(0), rows = grad_y.numel() / outputs;
    if (!one_launch(rows, inputs, outputs, type, need_x, need_bias)) return false;
    const Tensor x = x_of();
    if (!in_memory(x, type, device) || x.numel() != rows * inputs) return false;
    out.weight = empty_on(weight, {outputs, inputs}, type);
    if (need_bias) out.bias = empty_on(weight, {outputs}, type);
    if (need_x) {
        std::vector<int64_t> shape = grad_y.sizes().vec();
        shape.back() = inputs;
        out.x = empty_on(grad_y, shape, type);
    }
    const auto pointer = [](const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; };
    call(api.linear_backward, pointer(grad_y), pointer(weight), pointer(x), dtype_of(grad_y), rows, inputs, outputs, pointer(out.x), pointer(out.weight),
         pointer(out.bias), current_stream());
    return true;
}

// (rows, inputs, outputs, whether binary16, whether x and bias need theirs beside the weight) -> whether the rule is for the launch
PyObject* linear_one_launch_impl(PyObject* const* a)
{
    return PyBool_FromLong(one_launch(integer(a[0]), integer(a[1]), integer(a[2]), a[3] == Py_True ? at::kHalf : at::kFloat, a[4] == Py_True, a[5] == Py_True));
}
ACTQ_ENTRY(linear_one_launch, 6)

// (grad_y, weight, x, whether x, weight, bias need theirs) -> their gradients (None where none is needed), or None if torch's operators have to serve
PyObject* linear_gradients_impl(PyObject* const* a)
{
    const Tensor &grad_y = tensor_of(a[0], "grad_y"), &weight = tensor_of(a[1], "weight"), &x = tensor_of(a[2], "x");
    LinearGradients g;
    if (x.dim() < 1 || !fused_gradients(grad_y, weight, [&] { return x; }, x.scalar_type(), x.size(-1), a[3] == Py_True, a[4] == Py_True, a[5] == Py_True, g))
        Py_RETURN_NONE;
    const auto wrap = [](const Tensor& t) {
        if (t.defined()) return THPVariable_Wrap(t);
        Py_INCREF(Py_None);
        return Py_None;
    };
    return tuple_of({wrap(g.x), wrap(g.weight), wrap(g.bias)});
}
ACTQ_ENTRY(linear_gradients, 6)

// The activation-compressed linear layer: the saved input is the compressed one.
struct LinearFn : torch::autograd::Function<LinearFn> {
    static Tensor forward(AutogradContext* ctx, const Tensor& x, const Tensor& weight, const std::optional<Tensor>& bias, const Config& config)
    {
        const Compressed c = compress_activation(x.contiguous(), std::nullopt, config);
        ctx->save_for_backward({c.bits, c.offsets, c.packed, c.header, weight});
        ctx->saved_data["shape"] = x.sizes().vec();
        ctx->saved_data["half"] = x.scalar_type() == at::kHalf;
        ctx->saved_data["bias"] = bias.has_value();
        ctx->saved_data["hf"] = config.hf;
        return at::linear(x, weight, bias);
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads)
    {
        const variable_list saved = ctx->get_saved_variables();
        const Tensor &bits = saved[0], &offsets = saved[1], &packed = saved[2], &header = saved[3], &weight = saved[4];
        const Tensor& grad_y = grads[0];
        const std::vector<int64_t> shape = ctx->saved_data["shape"].toIntVector();
        const at::ScalarType type = ctx->saved_data["half"].toBool() ? at::kHalf : at::kFloat;
        const int64_t hf = ctx->saved_data["hf"].toInt();
        // under autocast the output (and so grad_y) is narrower than the saved input and the weight: the stock backward
        // then computes in grad_y's type and returns gradients of the operands' types
        const at::ScalarType ct = grad_y.scalar_type();
        const bool need_bias = ctx->saved_data["bias"].toBool() && ctx->needs_input_grad(2);
        Tensor x;
        const auto decompressed = [&] {
            if (!x.defined()) {
                x = empty_on(bits, shape, type);
                decompress(packed, header, bits, offsets, x, view_of(x), kG, hf, nullptr);
            }
            return x;
        };
        LinearGradients g;
        if (fused_gradients(grad_y, weight, decompressed, type, shape.back(), ctx->needs_input_grad(0), ctx->needs_input_grad(1), need_bias, g))
            return {g.x, g.weight, g.bias, Tensor()};
        const Tensor g2 = grad_y.reshape({-1, grad_y.size(-1)});
        Tensor grad_x, grad_w, grad_b;
        if (ctx->needs_input_grad(0)) grad_x = grad_y.matmul(weight.to(ct)).to(type);
        if (ctx->needs_input_grad(1)) grad_w = g2.t().matmul(decompressed().reshape({-1, shape.back()}).to(ct)).to(weight.scalar_type());
        if (need_bias) grad_b = g2.sum(0).to(weight.scalar_type());
        return {grad_x, grad_w, grad_b, Tensor()};
    }
};

// Exact: the context is one bit per element.
struct ReluFn : torch::autograd::Function<ReluFn> {
    static Tensor forward(AutogradContext* ctx, const Tensor& input)
    {
        const Tensor x = input.contiguous();
        const Tensor y = at::empty_like(x), mask = empty_on(x, {mask_bytes(x.numel())}, at::kByte);
        relu_forward_call(x, y, mask, nullptr);
        ctx->save_for_backward({mask});
        return y;
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads)
    {
        const Tensor mask = ctx->get_saved_variables()[0], grad_y = grads[0].contiguous();
        const Tensor grad_x = at::empty_like(grad_y);
        relu_backward_call(mask, grad_y, grad_x, nullptr);
        return {grad_x};
    }
};

// Exact: the context is the 8-bit window position of every output location.
struct MaxPoolFn : torch::autograd::Function<MaxPoolFn> {
    static Tensor forward(AutogradContext* ctx, const Tensor& input, const Window& w)
    {
        const Tensor x = input.contiguous();
        const Pooling p = pooling_of(x, w);
        const std::vector<int64_t> shape = with_extent(x, p.OH, p.OW);
        const Tensor y = empty_on(x, shape, x.scalar_type()), arg = empty_on(x, shape, at::kByte);
        maxpool_forward_call(x, p, w, y, arg, nullptr);
        ctx->save_for_backward({arg});
        ctx->saved_data["geometry"] = std::vector<int64_t>{p.H, p.W, w.k[0], w.k[1], w.s[0], w.s[1], w.p[0], w.p[1], w.d[0], w.d[1]};
        return y;
    }

    static variable_list backward(AutogradContext* ctx, variable_list grads)
    {
        const Tensor arg = ctx->get_saved_variables()[0], grad_y = grads[0].contiguous();
        const std::vector<int64_t> g = ctx->saved_data["geometry"].toIntVector();
        Window w;
        for (int i = 0; i < 2; ++i) {
            w.k[i] = static_cast<int32_t>(g[2 + i]);
            w.s[i] = static_cast<int32_t>(g[4 + i]);
            w.p[i] = static_cast<int32_t>(g[6 + i]);
            w.d[i] = static_cast<int32_t>(g[8 + i]);
        }
        const Pooling p = pooling_of_gradient(grad_y, static_cast<int32_t>(g[0]), static_cast<int32_t>(g[1]), w);
        const Tensor grad_x = empty_on(grad_y, with_extent(grad_y, p.H, p.W), grad_y.scalar_type());
        maxpool_backward_call(arg, grad_y, p, w, grad_x, nullptr);
        return {grad_x, Tensor()};
    }
};

template <typename F>
PyObject* without_gil(F f)
{
    Tensor y;
    {
        pybind11::gil_scoped_release no_gil;
        y = f();
    }
    return THPVariable_Wrap(y);
}

// (x, weight, bias or None, then config_of's nine) -> y
PyObject* linear_impl(PyObject* const* a)
{
    const Tensor x = tensor_of(a[0], "x"), weight = tensor_of(a[1], "weight");
    const std::optional<Tensor> bias = optional_tensor(a[2], "bias");
    const Config config = config_of(a + 3);
    return without_gil([&] { return LinearFn::apply(x, weight, bias, config); });
}
ACTQ_ENTRY(linear, 12)

// (x) -> y
PyObject* relu_impl(PyObject* const* a)
{
    const Tensor x = tensor_of(a[0], "x");
    return without_gil([&] { return ReluFn::apply(x); });
}
ACTQ_ENTRY(relu, 1)

// (x, kernel, stride, padding, dilation) -> y
PyObject* maxpool2d_impl(PyObject* const* a)
{
    const Tensor x = tensor_of(a[0], "x");
    const Window w = window_of(a + 1);
    return without_gil([&] { return MaxPoolFn::apply(x, w); });
}
ACTQ_ENTRY(maxpool2d, 5)

// True if nothing is active that watches or transforms Python-level autograd functions: torch.jit tracing, functorch's
// transforms, torch-function modes, tensor subclasses, tangents of forward-mode differentiation.  The layers then
// take the functions of this file; otherwise those written in Python.
PyObject* plain(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    bool ok = !torch::jit::tracer::isTracing() && !at::impl::torch_function_mode_enabled() &&
              !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
    for (Py_ssize_t i = 0; ok && i < n; ++i)
        ok = a[i] == Py_None || (THPVariable_CheckExact(a[i]) && !THPVariable_Unpack(a[i])._fw_grad(0).defined());
    return PyBool_FromLong(ok);
    END_HANDLE_TH_ERRORS
}

// (exception class, addresses in the order of Api)
PyObject* attach_impl(PyObject* const* a)
{
    constexpr Py_ssize_t kEntries = sizeof(Api) / sizeof(void*);
    TORCH_CHECK_TYPE(PyTuple_Check(a[1]) && PyTuple_GET_SIZE(a[1]) == kEntries, "attach takes ", kEntries, " addresses");
    void* address[kEntries];
    for (Py_ssize_t i = 0; i < kEntries; ++i) {
        address[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[1], i));
        if (PyErr_Occurred()) throw python_error();
        TORCH_CHECK_VALUE(address[i] != nullptr, "attach: null address");
    }
    static_assert(sizeof(address) == sizeof(Api), "one address per entry");
    std::memcpy(&api, address, sizeof(Api));
    Py_INCREF(a[0]);
    Py_XSETREF(actq_error, a[0]);
    Py_RETURN_NONE;
}
ACTQ_ENTRY(attach, 2)

#define ACTQ_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ACTQ_METHOD(attach), ACTQ_METHOD(plain), ACTQ_METHOD(group_stats), ACTQ_METHOD(sample_sensitivity), ACTQ_METHOD(allocate_bits_device),
    ACTQ_METHOD(quantize_pack), ACTQ_METHOD(unpack_dequantize), ACTQ_METHOD(compress_mixed), ACTQ_METHOD(relu_forward), ACTQ_METHOD(relu_backward),
    ACTQ_METHOD(maxpool2d_forward), ACTQ_METHOD(maxpool2d_backward), ACTQ_METHOD(linear_one_launch), ACTQ_METHOD(linear_gradients), ACTQ_METHOD(linear), ACTQ_METHOD(relu), ACTQ_METHOD(maxpool2d),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "actq_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

#ifndef ACTQ_SOURCE_HASH
#define ACTQ_SOURCE_HASH "unknown"
#endif
// the digest follows a fixed marker, so that it can be read from the file without loading it
const char source_digest[] = "actq-source-digest:" ACTQ_SOURCE_HASH;

}  // namespace

PyMODINIT_FUNC PyInit_actq_torch(void)
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "source_hash", source_digest + sizeof("actq-source-digest:") - 1) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
