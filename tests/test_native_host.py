"""The native module of the binding: built from the source beside it, and left alone where something watches or
transforms Python-level autograd functions (nothing here touches a GPU)."""
import pytest
import torch
import torch.autograd.forward_ad as forward_ad
import torch.nn as nn

from paper_2104_14129_amd import binding as B
from paper_2104_14129_amd import build as lib_build
from paper_2104_14129_amd import layers as L


def test_the_native_module_was_built_from_the_source_beside_it():
    assert B.host().source_hash == lib_build.host_source_hash() == B._digest_in_file(B.HOST_PATH)


def test_plain_tensors_and_parameters_take_the_native_functions():
    x = torch.randn(3, 4)
    assert L._native(x) and L._native(x.requires_grad_(), nn.Parameter(x.detach()), None)
    with torch.no_grad():
        assert L._native(x)


class _Watching(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("what", ["trace", "vmap", "grad", "jvp", "dual", "mode", "subclass", "no tensor"])
def test_watched_tensors_take_the_functions_in_python(what):
    x, seen = torch.randn(3, 4), []

    def probe(t):
        seen.append(L._native(t))
        return (t * 1.0).sum()

    if what == "trace":
        torch.jit.trace(probe, x, check_trace=False)
    elif what == "vmap":
        torch.func.vmap(probe)(x)
    elif what == "grad":
        torch.func.grad(probe)(x)
    elif what == "jvp":
        torch.func.jvp(probe, (x,), (x,))
    elif what == "dual":
        with forward_ad.dual_level():
            probe(forward_ad.make_dual(x, x))
    elif what == "mode":
        with _Watching():
            seen.append(L._native(x))
    elif what == "subclass":
        seen.append(L._native(x.as_subclass(_Sub)))
    else:
        seen.append(L._native(x.numpy()))
    assert seen == [False]


@pytest.mark.parametrize("what,kind,call", [
    ("one dimension", IndexError, lambda h: h.maxpool2d(torch.randn(5), (2, 2), (2, 2), (0, 0), (1, 1))),
    ("no dimension", IndexError, lambda h: h.maxpool2d(torch.tensor(1.0), (2, 2), (2, 2), (0, 0), (1, 1))),
    ("no rows", ZeroDivisionError, lambda h: h.maxpool2d(torch.randn(2, 0, 5), (2, 2), (2, 2), (0, 0), (1, 1))),
    ("no columns", ZeroDivisionError, lambda h: h.maxpool2d(torch.randn(2, 5, 0), (2, 2), (2, 2), (0, 0), (1, 1))),
    ("window too large", B.ActqError, lambda h: h.maxpool2d(torch.randn(2, 4, 4), (9, 9), (2, 2), (0, 0), (1, 1))),
    ("no samples", ZeroDivisionError, lambda h: h.linear(torch.randn(0, 5), torch.randn(3, 5), None, 100, 0x116, 64, 1, 1, 16, 0, None, None)),
])
def test_errors_of_the_autograd_functions_are_python_exceptions(what, kind, call):
    """The functions run without the interpreter's lock; what they refuse is raised with it, once and again."""
    for _ in range(2):
        with pytest.raises(kind):
            call(B.host())
    with pytest.raises(ValueError, match="GPU"):     # and the next call is served as usual
        B.host().relu(torch.randn(3))


@pytest.mark.parametrize("G,kind", [(0, ZeroDivisionError), (-1, ValueError), (-256, ValueError), (2 ** 31, ValueError), (2 ** 32 + 256, ValueError)])
def test_a_group_size_that_is_none_is_refused(G, kind):
    """Before anything is divided by it, and before a size beyond 32 bits becomes another one on its way to the library."""
    x, bits, offsets = torch.randn(4, 512), torch.full((4,), 2, dtype=torch.uint8), torch.arange(4) * 128
    packed, header = torch.zeros(512, dtype=torch.uint8), torch.zeros(16)
    for call in (lambda: B.group_stats(x, G=G), lambda: B.quantize_pack(x, bits, offsets, packed, header, 1, G=G),
                 lambda: B.unpack_dequantize(packed, header, bits, offsets, x, G=G)):
        with pytest.raises(kind, match="^G must"):
            call()


@pytest.mark.parametrize("shape", [(1, 2 ** 32 + 4, 2), (1, 2, 2 ** 32 + 4), (2 ** 31, 1)])
def test_pooling_extents_beyond_32_bits_are_refused(shape):
    """2^32 + 4 rows are not 4, in the functions that allocate by the one and count planes by the other."""
    x, window = torch.empty(shape, dtype=torch.float16, device="meta"), ((1, 1), (1, 1), (0, 0), (1, 1))
    grad = torch.empty((1, 4, 4), dtype=torch.float16, device="meta")
    for call in (lambda: B.host().maxpool2d(x, *window), lambda: B.maxpool2d_forward(x, *window),
                 lambda: B.maxpool2d_backward(grad, grad, *shape[-2:], *window)):
        with pytest.raises(ValueError, match="fit 32 bits"):
            call()


@pytest.mark.parametrize("native", [True, False])
def test_a_parametrized_weight_is_computed_once_per_forward_pass(native, monkeypatch):
    """A parametrization may keep state (spectral normalization steps its power iteration in each evaluation)."""
    class Counting(nn.Module):
        evaluations = 0

        def forward(self, w):
            self.evaluations += 1
            return w * 1.0

    class OnGpu:     # as much of a tensor as the layer looks at before it hands it on
        is_cuda, dtype, shape, device = True, torch.float32, torch.Size((3, 4)), torch.device("cpu")

        def numel(self):
            return 12

    class Host:
        def linear(self, x, weight, bias, *settings):
            return weight, bias

    m, counting, seen = L.QLinear(4, 2), Counting(), []
    nn.utils.parametrize.register_parametrization(m, "weight", counting, unsafe=True)
    counting.evaluations = 0
    monkeypatch.setattr(L, "_native", lambda *t: seen.append(t[1]) or native)
    monkeypatch.setattr(B, "_host", Host())
    monkeypatch.setattr(L._QLinearFn, "apply", lambda x, weight, bias: (weight, bias))
    weight, bias = m(OnGpu())
    assert counting.evaluations == 1 and weight is seen[0] and bias is m.bias


@pytest.mark.parametrize("what", ["interpreter", "torch", "C++ library"])
def test_the_digest_names_all_that_the_module_is_built_against(what, monkeypatch):
    import sysconfig
    before, stock = lib_build.host_source_hash(), sysconfig.get_config_var
    if what == "interpreter":
        monkeypatch.setattr(sysconfig, "get_config_var", lambda name: "cpython-399-x86_64-linux-gnu" if name == "SOABI" else stock(name))
    elif what == "torch":
        monkeypatch.setattr(torch, "__version__", "0.0.0")
    else:
        monkeypatch.setattr(torch._C, "_GLIBCXX_USE_CXX11_ABI", not torch._C._GLIBCXX_USE_CXX11_ABI)
    assert lib_build.host_source_hash() != before
