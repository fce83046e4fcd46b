"""The eager calls in native code (csrc/bl_calls.cpp) beside the Python path that they stand in for."""
import copy

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_16144_amd import binding as B      # noqa: E402
from paper_2410_16144_amd import decoder, ops      # noqa: E402


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _weight(dev, N, K, seed=5):
    w = torch.randint(-1, 2, (N, K), dtype=torch.int8, device=dev, generator=torch.Generator(dev).manual_seed(seed))
    return ops.pack_ternary(w, 0.02)


def _with_desc(pw, **fields):
    desc = copy.copy(pw.desc)
    for k, v in fields.items():
        setattr(desc, k, v)
    return ops.PackedWeight(pw.blob, desc)


def test_a_status_is_raised_and_the_call_is_not_repeated(dev, monkeypatch):
    """The library refuses the call: its status is raised from the native call's own answer, and the ctypes binding, which
    would make the call a second time, is not reached."""
    pw = _weight(dev, 128, 256)
    x = torch.randn(4, 256, device=dev)
    qa = ops.quant_act(x)
    nine = ops.quant_act(torch.randn(9, 256, device=dev))
    long_h = torch.zeros((1, B.BL_NORM_MAX_K + 4), device=dev)
    torch.cuda.synchronize()

    def again(name):
        def called(*a, **k):
            raise AssertionError(name + " called a second time")
        return called
    for name in ("bl_quant_act", "bl_gemv", "bl_gemm", "bl_gemm_batch", "bl_norm_quant"):
        monkeypatch.setattr(B, name, again(name))
    for what, status, call in (
            ("bl_quant_act", B.BL_ERR_SHAPE, lambda: ops.quant_act(x[:1].expand(3, 256))),              # rows closer than K
            ("bl_gemv", B.BL_ERR_M_RANGE, lambda: ops.gemv(pw, nine)),
            ("bl_gemv", B.BL_ERR_BUF_SMALL, lambda: ops.gemv(_with_desc(pw, bytes=64), qa)),
            ("bl_gemm", B.BL_ERR_LAYOUT, lambda: ops.gemm(_with_desc(pw, version=7), qa)),
            ("bl_gemm_batch", B.BL_ERR_LAYOUT, lambda: ops.gemm_batch([pw, _with_desc(pw, version=7)], qa)),
            ("bl_norm_quant", B.BL_ERR_SHAPE, lambda: decoder.norm_quant(B.BL_NORM_RESIDUAL, long_h[0].clone(), h=long_h))):
        with pytest.raises(B.BitLinearError) as e:
            call()
        assert e.value.status == status and what + " failed" in str(e.value)


def test_prepared_launches_refuse_and_take_what_the_binding_does(dev):
    """Items that are not the launch's ctypes array: none at all and another launch's raise, an iterable of tuples is launched."""
    pw = _weight(dev, 128, 256)
    qa = ops.quant_act(torch.randn(1, 256, device=dev))
    group = ops.GemvGroup([pw], [qa])
    want = group.launch()[0].clone()
    row = (pw.blob.data_ptr(), pw.desc, qa.q.data_ptr(), qa.a_scale.data_ptr(), qa.q_sum.data_ptr(), group.outs[0].data_ptr(), 0)
    for items in ([row], iter([row]), B.make_gemv_items([row])):
        group.outs[0].fill_(-1.0)
        group.items = items
        assert torch.equal(group.launch()[0], want)
    group.workspace_ptr = None      # as 0: no workspace
    group.outs[0].fill_(-1.0)
    group.items = B.make_gemv_items([row])
    assert torch.equal(group.launch()[0], want)
    import ctypes
    for items in ([], B.make_gemv_items([])):
        group.items = items
        with pytest.raises(B.BitLinearError) as e:
            group.launch()
        assert e.value.status == B.BL_ERR_COUNT
    group.items = B.make_quant_items([])
    with pytest.raises(ctypes.ArgumentError):
        group.launch()


def test_the_native_module_is_the_one_that_runs(dev):
    assert B.calls() and B.calls().__file__ == __import__("paper_2410_16144_amd.build", fromlist=["build"]).calls_path()


def test_every_function_gives_the_same_without_the_native_module(dev, monkeypatch):
    """Both paths over the same inputs: same bits, same types."""
    pw, pw2 = _weight(dev, 200, 260), _weight(dev, 70, 260, 6)
    x = torch.randn(11, 260, device=dev)
    a, b, h = (torch.randn(11, 260, device=dev) for _ in range(3))
    gamma = torch.rand(260, device=dev) + 0.5

    def everything():
        qa = ops.quant_act(x)
        qb = ops.quant_act(x.bfloat16(), ops.alloc_quant(11, 260, dev))
        few = ops.quant_act(x[:3])
        y = torch.empty_like(a)
        assert decoder.norm_quant(B.BL_NORM_PLAIN, gamma, a=a, y=y, quantize=False) is None
        hh = h.clone()
        n = [decoder.norm_quant(B.BL_NORM_GATED, gamma, a=a, b=b), decoder.norm_quant(B.BL_NORM_RESIDUAL, gamma, a=a, h=hh)]
        acc = ops.gemm(pw, qa, want_acc=True)
        group = ops.GemvGroup([pw, pw2], [few, few])
        outs = [ops.gemm(pw, qa), ops.gemv(pw2, few), *acc, *ops.gemm_batch([pw, pw2], qa), *group.launch(), y, hh]
        return outs + [t for q in (qa, qb, few, *n) for t in (q.q, q.a_scale, q.q_sum)] + [torch.tensor([q.K for q in (qa, qb, *n)])]

    native = everything()
    monkeypatch.setattr(B, "_calls", False)
    for one, other in zip(native, everything()):
        assert one.dtype == other.dtype and torch.equal(one, other)


class Plain(torch.Tensor):
    """A subclass without a say of its own."""


class Loud(torch.Tensor):
    """A subclass that sees every torch function."""
    seen = []

    @classmethod
    def __torch_function__(cls, func, types, args=(), kwargs=None):
        Loud.seen.append(getattr(func, "__name__", str(func)))
        return super().__torch_function__(func, types, args, kwargs or {})


class Watch(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        Loud.seen.append(getattr(func, "__name__", str(func)))
        return func(*args, **(kwargs or {}))


def _watched(call):
    with Watch():
        return call()


def _outcome(call):
    """What a call gives or raises, comparable."""
    try:
        r = call()
    except Exception as e:      # noqa: BLE001 -- the kind and the words are what is compared
        return type(e).__name__, str(e)
    torch.cuda.synchronize()
    r = r if isinstance(r, (list, tuple)) else [r]
    flat = [t for q in r for t in ((q.q, q.a_scale, q.q_sum) if isinstance(q, ops.QuantAct) else (q,))]
    return [None if t is None else (t.dtype, t.shape, t.cpu().contiguous().view(torch.uint8).numpy().tobytes()) for t in flat]


@pytest.mark.parametrize("inference", [False, True])
def test_fresh_outputs_are_what_torch_allocates(dev, monkeypatch, inference):
    """Outputs come straight from the allocator: the same kind of tensors as torch.empty's, in inference mode too."""
    pw = _weight(dev, 100, 256)
    x = torch.randn(3, 256, device=dev)

    def outputs():
        with torch.inference_mode(inference):
            qa = ops.quant_act(x)
            return [qa.q, qa.a_scale, qa.q_sum, *ops.gemv(pw, qa, want_acc=True), *ops.gemm_batch([pw, pw], qa)]
    native = outputs()
    monkeypatch.setattr(B, "calls", lambda: None)
    for a, b in zip(native, outputs(), strict=True):
        assert torch.equal(a, b)
        for what in (lambda t: t.is_inference(), lambda t: t.requires_grad, lambda t: t.dtype, lambda t: t.device, lambda t: t.stride(),
                     lambda t: t.untyped_storage().nbytes(), lambda t: t.storage_offset(), lambda t: t.layout, lambda t: type(t)):
            assert what(a) == what(b)


def test_what_the_native_calls_refuse_ends_as_without_them(dev, monkeypatch):
    """Operands that are not plain device tensors of the expected kind: the same result, or the same error, as by ctypes."""
    g = torch.Generator(dev).manual_seed(3)
    pw = _weight(dev, 96, 128)
    x, a, b = (torch.randn((5, 128), device=dev, generator=g) for _ in range(3))
    h, gamma = torch.randn((5, 128), device=dev, generator=g), torch.rand(128, device=dev, generator=g) + 0.5
    qa = ops.quant_act(x)
    norm = lambda **k: decoder.norm_quant(k.pop("mode", B.BL_NORM_GATED), k.pop("gamma", gamma), **{"a": a, "b": b, **k})
    calls = {
        "half": lambda: ops.quant_act(x.half()), "double": lambda: ops.quant_act(x.double()), "cpu": lambda: ops.quant_act(x.cpu()),
        "one dimension": lambda: ops.quant_act(x[0]), "transposed": lambda: ops.quant_act(x.t()), "strided rows": lambda: ops.quant_act(x[:, :100]),
        "no rows": lambda: ops.quant_act(x[:0]), "subclass": lambda: ops.quant_act(x.as_subclass(Plain)),
        "loud subclass": lambda: ops.quant_act(x.as_subclass(Loud)), "parameter": lambda: ops.quant_act(torch.nn.Parameter(x)),
        "a mode": lambda: _watched(lambda: ops.quant_act(x)), "a mode over a product": lambda: _watched(lambda: ops.gemm(pw, qa)),
        "vmap": lambda: torch.func.vmap(lambda r: ops.quant_act(r).a_scale)(x.view(5, 1, 128)),
        "grad": lambda: torch.func.grad(lambda r: ops.quant_act(r).a_scale.sum())(x),
        "sparse": lambda: ops.quant_act(x.to_sparse()),
        "too many rows": lambda: ops.gemv(pw, ops.quant_act(x.repeat(3, 1))), "no token": lambda: ops.gemm(pw, ops.QuantAct(qa.q[:0], qa.a_scale, qa.q_sum, 128)),
        "another layout": lambda: ops.gemm(_with_desc(pw, version=9), qa),
        "another K": lambda: ops.gemm(_with_desc(pw, K=64), qa),
        "batch of another layout": lambda: ops.gemm_batch([pw, _with_desc(pw, version=2)], qa),
        "norm of half": lambda: norm(a=a.half()), "norm of a slice": lambda: norm(a=a[:, :64], b=b[:, :64], gamma=gamma[:64].clone()),
        "norm of strided rows": lambda: norm(a=torch.cat([a, a], 1)[:, :128]), "norm of other rows": lambda: norm(b=b[:4]),
        "norm without a gate": lambda: norm(b=None), "norm weight of another length": lambda: norm(gamma=gamma[:64].clone()),
        "norm weight of two dimensions": lambda: norm(gamma=gamma[None]), "norm weight of half": lambda: norm(gamma=gamma.half()),
        "little scratch": lambda: norm(scratch=torch.empty(16, dtype=torch.uint8, device=dev)),
        "norm of a subclass": lambda: norm(a=a.as_subclass(Plain)), "no such mode": lambda: norm(mode=9),
        "residual without a delta": lambda: [norm(mode=B.BL_NORM_RESIDUAL, a=None, b=None, h=h.clone())],
        "norm with integer eps": lambda: norm(eps=1), "norm with an eps of text": lambda: norm(eps="x"),
    }
    native = {}
    for name, call in calls.items():
        Loud.seen.clear()
        native[name] = _outcome(call), list(Loud.seen)
    monkeypatch.setattr(B, "_calls", False)
    for name, call in calls.items():
        Loud.seen.clear()
        assert native[name] == (_outcome(call), list(Loud.seen)), name
