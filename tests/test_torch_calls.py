"""The native calls behind binding.py's per-step functions take the plain case only and leave the rest, errors included, to
the Python way (no GPU needed for what they refuse)."""
import os

import pytest
import torch

import paper_2302_03213_amd as lut
from paper_2302_03213_amd import binding


def layer():
    return lut.LutLayer(torch.zeros((2, 16, 4)), torch.zeros((2, 16, 8)), lut.TABLE_F32, 8)


def test_tensors_that_are_not_on_the_gpu_are_left_alone():
    l, X = layer(), torch.zeros((3, 8))
    calls = binding._calls
    assert calls.linear(l.address, X) is None and calls.linear(l.address, l.address, X) is None
    assert calls.linear(l.address, None) is None and calls.linear(l.address) is None
    assert calls.linear_tree16(l.address, l.address, X) is None
    assert calls.conv2d(l.address, torch.zeros((1, 2, 2, 2)), 1, 1, 0) is None
    assert calls.build_table(torch.zeros((2, 16, 4)), torch.zeros((8, 8)), 0) is None
    assert calls.linear_gradient(X, X) is None
    assert calls.softpq_backward(torch.zeros((2, 16, 4)), 8, 1.0, X, X, True) is None
    assert calls.softpq_backward_conv2d(torch.zeros((2, 16, 4)), 1.0, X, X, X, True, 1, 1, 0) is None
    with pytest.raises(AssertionError):
        lut.linear(l, X)
    with pytest.raises(AssertionError):
        lut.conv2d(l, torch.zeros((1, 2, 2, 2)), 1)


def test_the_file_is_bound_to_torch_and_the_interpreter(monkeypatch):
    build, is_current = binding._build, binding._is_current
    made = build.torch_calls_hash()
    assert is_current(build.TORCH_CALLS, made) and not is_current(build.TORCH_CALLS + ".gone", made)
    monkeypatch.setattr(torch, "__version__", "2.11.0")
    assert not is_current(build.TORCH_CALLS, build.torch_calls_hash())
    monkeypatch.undo()
    monkeypatch.setattr(build.sysconfig, "get_config_var", lambda name: "cpython-313-x86_64-linux-gnu")
    assert not is_current(build.TORCH_CALLS, build.torch_calls_hash())


def test_headers_are_found_for_a_compiler_on_the_path(monkeypatch):
    monkeypatch.setenv("PATH", os.path.dirname(binding._build.HIPCC), prepend=os.pathsep)
    monkeypatch.setattr(binding._build, "HIPCC", "hipcc")
    assert os.path.exists(os.path.join(binding._build._rocm_include(), "hip", "hip_runtime.h"))


def test_without_a_compiler_everything_takes_the_python_way(monkeypatch, tmp_path):
    def fails():
        raise RuntimeError("no g++")
    monkeypatch.setattr(binding._build, "TORCH_CALLS", str(tmp_path / "torch_calls.so"))
    monkeypatch.setattr(binding._build, "build_torch_calls", fails)
    with pytest.warns(UserWarning, match="no g[+][+]"):
        calls = binding._load_torch_calls()
    assert calls.linear(1, 2) is None and calls.bias_gradient(3) is None


@pytest.mark.gpu
def test_what_was_refused_is_refused_and_forms_agree():
    P, W = torch.randn((6, 16, 4), device="cuda"), torch.randn((24, 40), device="cuda")
    l = lut.build_table(P, W, lut.TABLE_I8)
    X = torch.randn((300, 24), device="cuda")
    ws = torch.empty((300, 6), dtype=torch.uint8, device="cuda")
    ref = lut.linear(l, X, idx_workspace=ws)
    wide = torch.randn((300, 31), device="cuda")
    wide[:, 3:27] = X
    for x in (X, wide[:, 3:27], torch.nn.Parameter(X), X.clone().requires_grad_(True)):
        got = lut.linear(l, x)
        assert torch.equal(got, ref) and not got.requires_grad
    for bad in (X.t(), X.double(), X.cpu(), X[0]):
        with pytest.raises((AssertionError, IndexError)):
            lut.linear(l, bad)
    with pytest.raises(lut.LutnnError):
        lut.linear(l, X[:, :20].contiguous())  # rows narrower than C * V
    with pytest.raises(ValueError):
        lut.build_table(P, W[:20], lut.TABLE_I8)
    with pytest.raises(ValueError):
        lut.conv2d(l, torch.randn((1, 24, 2, 2), device="cuda"), 5)
    image = torch.randn((2, 24, 5, 5), device="cuda")
    assert torch.equal(lut.conv2d(l, image, (1, 1), (2, 2), (0, 0)), lut.conv2d(l, image, 1, 2, 0))
    assert lut.linear(l, X[:0]).shape == (0, 40)


@pytest.mark.gpu
def test_where_tensors_give_no_pointers_the_python_way_reports_it():
    """Under torch.func.grad the outputs are wrappers without storage; under a dispatch mode their allocation can fail in
    Python: the exception leaves the native call with the interpreter's lock held and no error set."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Refuses(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise ValueError("refused")

    l = lut.build_table(torch.randn((6, 16, 4), device="cuda"), torch.randn((24, 40), device="cuda"), lut.TABLE_I8)
    X = torch.randn((300, 24), device="cuda")

    def inside(z):
        with pytest.raises(RuntimeError):
            lut.linear(l, X)
        return z.sum()

    torch.func.grad(inside)(torch.ones(3, device="cuda"))
    with Refuses(), pytest.raises(ValueError, match="refused"):
        lut.linear(l, X)
    assert lut.linear(l, X).shape == (300, 40)


def small_layers():
    """A layer per kind of call: (function of fresh inputs, its inputs)."""
    from paper_2302_03213_amd.softpq import SoftPQConv2d, SoftPQLinear
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    P, W = normal(12, 16, 4), normal(48, 40)
    tables = [lut.build_table(P, W, t) for t in (lut.TABLE_F32, lut.TABLE_I8, lut.TABLE_I4)]
    tree = lut.LutTree(torch.zeros((12, 15), dtype=torch.int32, device="cuda"), normal(12, 15), 4)
    deep = lut.LutTree(torch.zeros((12, 1023), dtype=torch.int32, device="cuda"), normal(12, 1023), 4)
    deep_table = lut.build_table(normal(12, 1024, 4), W, lut.TABLE_I8)

    def step(layer, x):
        x = x.detach().requires_grad_(True)
        Y = layer(x)
        return (Y.detach(),) + torch.autograd.grad(Y.square().sum(), (x, layer.centroids, layer.temperature, layer.bias))

    linear, conv = SoftPQLinear(P, W, bias=normal(40)), SoftPQConv2d(P, W, 2, 1, 1, bias=normal(40))
    return [(lambda x: [lut.linear(t, x) for t in tables], normal(300, 48)), (lambda x: lut.linear_tree(tables[1], tree, x), normal(2000, 48)),
            (lambda x: lut.linear_tree16(deep_table, deep, x), normal(100, 48)), (lambda x: lut.conv2d(tables[1], x, 2, 1, 1), normal(3, 12, 9, 9)),
            (lambda x: step(linear, x), normal(500, 48)), (lambda x: step(conv, x), normal(3, 12, 9, 9))]


def flat(outputs):
    return list(outputs) if isinstance(outputs, (list, tuple)) else [outputs]


@pytest.mark.gpu
def test_every_native_call_takes_the_plain_case_and_agrees_with_the_python_way(monkeypatch):
    taken, native = set(), binding._calls

    class Watched:
        def __getattr__(self, name):
            def call(*args):
                got = getattr(native, name)(*args)
                if got is not None:
                    taken.add(name)
                return got
            return call

    layers = small_layers()
    monkeypatch.setattr(binding, "_calls", Watched())
    got = [flat(f(x)) for f, x in layers]
    assert taken == {"linear", "linear_tree16", "conv2d", "build_table", "linear_gradient", "softpq_backward",
                     "softpq_backward_conv2d", "bias_gradient"}
    monkeypatch.setattr(binding, "_calls", binding._NoCalls())
    for (f, x), outputs in zip(layers, got):
        for a, b in zip(outputs, flat(f(x))):
            # torch's own sum stands for the bias gradient on the Python way
            assert torch.equal(a, b) or (a.shape == (40,) and torch.allclose(a, b, rtol=1e-5, atol=1e-4))


@pytest.mark.gpu
def test_other_streams_and_threads():
    """Each thread on a stream of its own: outputs and scratch come from that stream's memory."""
    import threading
    layers = small_layers()
    wanted = [[t.clone() for t in flat(f(x))] for f, x in layers]
    torch.cuda.synchronize()
    wrong = []

    def work(first):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for i in range(40):
                n = (first + i) % len(layers)
                f, x = layers[n]
                outputs = flat(f(x))
                stream.synchronize()
                if not all(torch.equal(a, b) for a, b in zip(outputs, wanted[n])):
                    wrong.append(n)

    threads = [threading.Thread(target=work, args=(n,)) for n in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
