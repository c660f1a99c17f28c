"""The calls that csrc/marshal.cpp takes over from Python: the same results bit for bit, the same refusals with
the same errors, and Python's own way wherever a tensor or a mode is not plain."""
import importlib.util
import subprocess
import sys
import types

import numpy as np
import pytest
import torch

from paper_2309_16119_amd import binding as b
from paper_2309_16119_amd import build, synth
from paper_2309_16119_amd.nn import ModuLoRALinear

gpu = pytest.mark.gpu


def test_the_module_is_built_for_this_torch():
    assert b._marshal is not None


@pytest.mark.parametrize("attribute", ["__version__", "git_version"])
def test_the_module_does_not_load_into_another_torch(attribute):
    """Another build of torch may have the same symbols and other class layouts: the import fails, and the binding does
    every call in Python."""
    code = ("import torch, torch.version; torch.version.%s = 'another'\n"
            "from paper_2309_16119_amd import binding as b; assert b._marshal is None\n"
            "import paper_2309_16119_amd._marshal") % attribute
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=build.ROOT)
    assert res.returncode != 0 and "ImportError: compiled for torch" in res.stderr, res.stderr[-500:]


@pytest.mark.parametrize("without", ["torch", "headers", "a_good_compile"])
def test_the_library_builds_without_the_module(monkeypatch, tmp_path, without):
    """libmodulora.so needs no torch: it is linked whether the module can be built or not, and no module of an earlier
    build stays behind where it cannot."""
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "SOURCES", ["optim.hip"])
    (tmp_path / "_marshal.so").write_text("stale")
    if without == "a_good_compile":
        def fails():
            raise RuntimeError("marshal.cpp does not compile")
        monkeypatch.setattr(build, "_build_marshal", fails)
        with pytest.raises(RuntimeError, match="marshal.cpp"):
            build.build_library()
    else:
        (tmp_path / "torch").mkdir()
        spec = None if without == "torch" else types.SimpleNamespace(origin=str(tmp_path / "torch" / "__init__.py"))
        monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: spec)
        build.build_library()
        assert not (tmp_path / "_marshal.so").exists()
    assert (tmp_path / "lib.so").exists()


def test_leaves_what_is_not_on_the_gpu_to_python():
    w = b.QWeight(torch.zeros(48, 256, dtype=torch.int32), torch.ones(4, 256, dtype=torch.float16),
                  torch.zeros(4, 256, dtype=torch.uint8), 512, 256, 3, 128)
    X, dY = torch.zeros(4, 512, dtype=torch.bfloat16), torch.zeros(4, 256, dtype=torch.bfloat16)
    A, B = torch.zeros(512, 8), torch.zeros(8, 256)
    assert b._marshal.product(False, False, w, X, A, B, 1.0, True) is None
    assert b._marshal.product(False, False, None, X, A, B, 1.0, True) is None
    assert b._marshal.gradients(False, X, dY, A, B, 1.0, None, None) is None
    assert b._marshal.layer(False, X, A, B, w, 1.0) is None
    assert b._marshal.product(False, False, w, "x", A, B, 1.0, True) is None
    with pytest.raises(AssertionError):
        b.modulora_fwd(w, X.float(), A, B, 1.0)
    with pytest.raises(AssertionError):
        b.modulora_bwd_lora(X, dY, A.t(), B, 1.0)


@pytest.mark.parametrize("marshal", [True, False])
def test_calls_of_two_threads_on_one_stream_do_not_overlap(monkeypatch, marshal):
    """A library call is several launches that share the stream's scratch memory, and Python's lock is released
    meanwhile: the next thread's call on that stream waits until the first has launched them all."""
    import threading
    import time

    log = []

    class Library:
        modulora_workspace_bytes = staticmethod(lambda *a: 64)

        @staticmethod
        def modulora_fwd(*a):
            log.append((threading.get_ident(), "first launch"))
            time.sleep(0.05)
            log.append((threading.get_ident(), "last launch"))
            return 0
    monkeypatch.setattr(b, "lib", Library)
    if not marshal:
        monkeypatch.setattr(b, "_marshal", None)
    monkeypatch.setattr(b, "_scratch_key", lambda device: (0, 12345), raising=False)
    monkeypatch.setattr(b, "_workspace", lambda device, nbytes: torch.empty(nbytes, dtype=torch.uint8))
    monkeypatch.setattr(b, "_stream", lambda: 0)
    w = b.QWeight(torch.zeros(48, 256, dtype=torch.int32), torch.ones(4, 256, dtype=torch.float16),
                  torch.zeros(4, 256, dtype=torch.uint8), 512, 256, 3, 128)
    X = torch.zeros(4, 512, dtype=torch.bfloat16)
    threads = [threading.Thread(target=lambda: [b.modulora_fwd(w, X, None, None, 1.0) for _ in range(2)]) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(log) == 12
    for first, last in zip(log[::2], log[1::2]):
        assert first == (last[0], "first launch") and last[1] == "last launch"

def _layer(f16, K=512, N=384, M=20, r=8, bits=3, group=128, seed=3):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, max(r, 1), seed=seed)
    L = synth.make_layer_torch(cfg, device="cuda", seed=seed)
    if f16:
        w = b.QWeightF16(L["qweight"], L["scales"], -L["scales"], torch.randn(N, device="cuda").half(), K, N, bits, group)
    else:
        w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
    dtype = torch.float16 if f16 else torch.bfloat16
    return w, L["X"].to(dtype), L["dY"].to(dtype), L["A"] if r else None, L["B"] if r else None


def _both(monkeypatch, call):
    """The call through marshal.cpp and through Python alone."""
    got = call()
    with monkeypatch.context() as m:
        m.setattr(b, "_marshal", None)
        ref = call()
    return got, ref


def _same(got, ref):
    if ref is None:
        assert got is None
        return
    assert got.dtype == ref.dtype and got.shape == ref.shape and got.device == ref.device and got.stride() == ref.stride()
    assert torch.equal(got.detach().view(torch.uint8), ref.detach().view(torch.uint8))


@gpu
@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("M,r", [(1, 8), (20, 8), (100, 3), (16, 0)])
def test_calls_return_what_python_does(monkeypatch, f16, M, r):
    w, X, dY, A, B = _layer(f16, M=M, r=r)
    fwd, bwd, grad = ((b.modulora_f16_fwd, b.modulora_f16_bwd_input, b.modulora_f16_bwd_lora) if f16 else
                      (b.modulora_fwd, b.modulora_bwd_input, b.modulora_bwd_lora))
    _same(fwd(w, X, A, B, "2")[0], fwd(w, X, A, B, 2.0)[0])          # float() is Python's to call
    for want in (True, False):
        for call in (lambda: fwd(w, X, A, B, 2, want_XA=want), lambda: bwd(w, dY, A, B, 2.0, want_dYBt=want)):
            got, ref = _both(monkeypatch, call)
            _same(got[0], ref[0])
            _same(got[1], ref[1])
    if r:
        XA, T = fwd(w, X, A, B, 2.0)[1], bwd(w, dY, A, B, 2.0)[1]
        for kw in (dict(), dict(XA=XA, dYBt=T)):
            got, ref = _both(monkeypatch, lambda: grad(X, dY, A, B, 2.0, **kw))
            _same(got[0], ref[0])
            _same(got[1], ref[1])
    if f16 and r:
        w.bias = None
        got, ref = _both(monkeypatch, lambda: fwd(w, X, A, B, 2.0))
        _same(got[0], ref[0])


@gpu
def test_refusals_are_pythons(monkeypatch):
    w, X, dY, A, B = _layer(False)
    odd = torch.zeros(20 * 512 + 4, dtype=torch.bfloat16, device="cuda")[4:].view(20, 512)     # eight bytes off
    bad = b.QWeight(w.qweight, w.scales, w.zeros, 512, 384, 5, 128)
    for call in (lambda: b.modulora_fwd(w, X.float(), A, B, 2.0), lambda: b.modulora_fwd(w, X[:, :256], A, B, 2.0),
                 lambda: b.modulora_fwd(w, X.t().contiguous().t(), A, B, 2.0), lambda: b.modulora_fwd(w, X, A.half(), B, 2.0),
                 lambda: b.modulora_fwd(w, X, A, B[:, :8], 2.0), lambda: b.modulora_fwd(w, odd, A, B, 2.0),
                 lambda: b.modulora_fwd(bad, X, A, B, 2.0), lambda: b.modulora_fwd(w, X[:0], A, B, 2.0),
                 lambda: b.modulora_bwd_lora(X, dY[:3], A, B, 2.0), lambda: b.modulora_fwd(w, X, A, B, "two"),
                 lambda: b.modulora_fwd(w, X.cpu(), A, B, 2.0), lambda: ModuLoRALinear(bad, r=0)(X)):
        errors = []
        for marshal in (b._marshal, None):
            with monkeypatch.context() as m, pytest.raises(Exception) as e:
                m.setattr(b, "_marshal", marshal)
                call()
            errors.append((type(e.value), str(e.value)))
        assert errors[0] == errors[1]


@gpu
@pytest.mark.parametrize("f16", [False, True])
def test_refused_backward_calls_are_pythons(monkeypatch, f16):
    """A gradient that is contiguous but eight bytes off: the same class, message and status from the backward pass."""
    w, X, dY, A, B = _layer(f16)
    module = ModuLoRALinear(w, r=8, alpha=16.0)
    odd = torch.zeros(20 * 384 + 4, dtype=dY.dtype, device="cuda")[4:].view(20, 384)
    spec = importlib.util.spec_from_file_location("paper_2309_16119_amd.binding_again", b.__file__)
    spec.loader.exec_module(importlib.util.module_from_spec(spec))       # another copy with a class of its own
    errors = []
    for marshal in (b._marshal, None):
        with monkeypatch.context() as m, pytest.raises(b.ModuloraError) as e:
            m.setattr(b, "_marshal", marshal)
            module(X.detach().requires_grad_(True)).backward(odd)
        errors.append((type(e.value), str(e.value), e.value.status))
    assert errors[0] == errors[1]


def _step(module, x, dy, inputs):
    y = module(x)
    return (y, *torch.autograd.grad(y, inputs, dy, allow_unused=True))


@gpu
@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("case", ["plain", "three_dims", "not_contiguous", "frozen_factors", "frozen_input", "no_adapter", "other_gradient_type"])
def test_module_returns_what_python_does(monkeypatch, f16, case):
    w, X, dY, A, B = _layer(f16, r=0 if case == "no_adapter" else 8)
    module = ModuLoRALinear(w, r=0 if A is None else 8, alpha=16.0)
    if A is not None:
        with torch.no_grad():
            module.A.copy_(A)
            module.B.copy_(B)
    x, dy = X, dY
    if case == "three_dims":
        x, dy = X.view(4, 5, -1), dY.view(4, 5, -1)
    if case == "not_contiguous":
        x, dy = X.t().contiguous().t(), dY.t().contiguous().t()
    x = x.detach().requires_grad_(case != "frozen_input")
    if case == "frozen_factors":
        module.A.requires_grad_(False)
        module.B.requires_grad_(False)
    inputs = [t for t in (x, module.A, module.B) if t is not None and t.requires_grad]
    if case == "other_gradient_type":
        got, ref = _both(monkeypatch, lambda: torch.autograd.grad(module(x).float().mul(0.5).sum(), inputs))
    else:
        got, ref = _both(monkeypatch, lambda: _step(module, x, dy, inputs))
        assert got[0].requires_grad and got[0].grad_fn is not None
    for g, r in zip(got, ref):
        _same(g, r)
    with torch.no_grad():
        y, yr = _both(monkeypatch, lambda: module(x))
    _same(y, yr)
    assert not y.requires_grad


@gpu
def test_module_keeps_pythons_ways(monkeypatch):
    """Saved-tensor hooks, checkpointing, in-place changes, a weight replaced between the passes, double backward,
    forward mode, vmap, tensor subclasses and dispatch modes."""
    from torch.utils._python_dispatch import TorchDispatchMode
    from torch.utils.checkpoint import checkpoint

    w, X, dY, A, B = _layer(False)
    module = ModuLoRALinear(w, r=8, alpha=16.0)
    with torch.no_grad():
        module.A.copy_(A)
        module.B.copy_(B)
    x = X.detach().requires_grad_(True)
    ins = (x, module.A, module.B)
    plain = _step(module, x, dY, ins)

    def hooked():
        seen = []
        with torch.autograd.graph.saved_tensors_hooks(lambda t: (seen.append(tuple(t.shape)), t.clone())[1], lambda t: t):
            y = module(x)
        return (seen, *torch.autograd.grad(y, ins, dY))
    got, ref = _both(monkeypatch, hooked)
    assert got[0] == ref[0] and len(got[0]) == 4
    for g, r, p in zip(got[1:], ref[1:], plain[1:]):
        _same(g, r)
        _same(g, p)
    for reentrant in (False, True):
        y = checkpoint(module, x, use_reentrant=reentrant)
        y.backward(dY)
        for t, p in zip(ins, plain[1:]):
            _same(t.grad, p)
            t.grad = None

    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        y = module(x)
        with torch.no_grad():
            module.A.mul_(1.0)
        y.backward(dY)
    # the frozen weight is read at the time of each pass
    def replaced():
        y = module(x)
        kept = w.scales
        w.scales = kept * 2
        try:
            return torch.autograd.grad(y, (x,), dY)
        finally:
            w.scales = kept
    got, ref = _both(monkeypatch, replaced)
    _same(got[0], ref[0])
    assert not torch.equal(got[0], plain[1])
    y = module(x)
    dx, = torch.autograd.grad(y, (x,), dY, create_graph=True)
    assert not dx.requires_grad

    for call in (lambda: torch.func.vmap(module)(X.view(4, 5, -1)),
                 lambda: torch.func.jvp(module, (X,), (X,))):
        errors = []
        for marshal in (b._marshal, None):
            with monkeypatch.context() as m, pytest.raises(Exception) as e:
                m.setattr(b, "_marshal", marshal)
                call()
            errors.append(type(e.value))
        assert errors[0] is errors[1]

    class Sub(torch.Tensor):
        pass
    assert b._marshal.layer(False, X.as_subclass(Sub), module.A, module.B, w, 2.0) is None

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert b._marshal.layer(False, X, module.A, module.B, w, 2.0) is None
        assert b._marshal.product(False, False, w, X, A, B, 2.0, True) is None


@gpu
def test_scratch_memory_per_stream_and_thread():
    """Calls of two threads on two streams at once, sizes that grow: each stream has its own buffer, and every
    result is that of the call alone."""
    import threading

    jobs = []
    for i in range(2):
        w, X, dY, A, B = _layer(False, K=1024, N=768, M=60 + 300 * i, seed=i)
        jobs.append((w, X, dY, A, B, b.modulora_fwd(w, X, A, B, 2.0)[0], b.modulora_bwd_input(w, dY, A, B, 2.0)[0]))
    torch.cuda.synchronize()
    failed = []

    def work(job, stream):
        w, X, dY, A, B, Y, dX = job
        with torch.cuda.stream(stream):
            for rows in (5, 40, X.shape[0]):
                b.modulora_fwd(w, X[:rows], A, B, 2.0)
            for _ in range(20):
                y, dx = b.modulora_fwd(w, X, A, B, 2.0)[0], b.modulora_bwd_input(w, dY, A, B, 2.0)[0]
                stream.synchronize()
                if not (torch.equal(y, Y) and torch.equal(dx, dX)):
                    failed.append(X.shape)
    threads = [threading.Thread(target=work, args=(job, torch.cuda.Stream())) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    device, first = torch.cuda.current_device(), torch.cuda.Stream()
    with torch.cuda.stream(first):
        a = b._workspace("cuda", 1000)
        assert b._workspace("cuda", 500).data_ptr() == a.data_ptr()
        grown = b._workspace("cuda", a.numel() + 1)
        assert grown.data_ptr() != a.data_ptr() and b._workspace("cuda", 10).data_ptr() == grown.data_ptr()
    assert b._workspace(torch.device("cuda", device), 0) is None


@gpu
@pytest.mark.parametrize("which", [0, 1, 2, 3])
@pytest.mark.parametrize("changed", [lambda t: t.t().contiguous().t(), lambda t: t.double(), lambda t: t[:-1].clone(), lambda t: t.cpu()])
def test_backward_refuses_other_tensors_from_hooks(which, changed):
    """What a saved-tensor hook brings back (activations, A, B, XA) is checked before anything is launched."""
    w, X, dY, A, B = _layer(False)
    module = ModuLoRALinear(w, r=8, alpha=16.0)
    x = X.detach().requires_grad_(True)
    count = []

    def pack(t):
        count.append(0)
        return len(count) - 1, t
    with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: changed(p[1]) if p[0] == which else p[1]):
        y = module(x)
    assert len(count) == 4
    with pytest.raises(RuntimeError, match="no longer what the forward pass saw"):
        torch.autograd.grad(y, (x, module.A, module.B), dY)


@gpu
@pytest.mark.parametrize("mixed", [False, True])
def test_scratch_memory_of_two_threads_on_one_stream(monkeypatch, mixed):
    """Calls of two threads on the same stream at once, of several launches each: every result is that of the call
    alone.  `mixed`: one of them with outputs given, which Python marshals."""
    import threading

    jobs = []
    for i, (K, N, M) in enumerate(((2048, 4096, 60), (4096, 2048, 300))):
        w, X, dY, A, B = _layer(False, K=K, N=N, M=M, seed=i)
        out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda") if mixed and i else None
        jobs.append((w, X, dY, A, B, b.modulora_fwd(w, X, A, B, 2.0)[0], b.modulora_bwd_input(w, dY, A, B, 2.0)[0], out))
    b.modulora_profile_begin()
    b.modulora_fwd(*jobs[0][:2], *jobs[0][3:5], 2.0)
    assert len(b.modulora_profile_end()) > 1
    torch.cuda.synchronize()
    failed = []

    def work(job):
        w, X, dY, A, B, Y, dX, out = job
        for _ in range(40):
            got = [(b.modulora_fwd(w, X, A, B, 2.0, out)[0].clone(), b.modulora_bwd_input(w, dY, A, B, 2.0)[0]) for _ in range(8)]
            torch.cuda.current_stream().synchronize()
            if not all(torch.equal(y, Y) and torch.equal(dx, dX) for y, dx in got):
                failed.append(X.shape)
    threads = [threading.Thread(target=work, args=(job,)) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
