"""The native module behind the binding (csrc/fc_torch.cpp): the ordinary call goes through it and gives what the checked
Python path of binding.py gives; everything else is left to that path."""
import sys
import threading
import warnings

import pytest

torch = pytest.importorskip("torch")

KINDS = ["asym", "sym", "fp8", "cmeta", "rot_asym", "rot_sym", "rot_fp8"]


class Declines:
    """stands in for the native module: takes no call"""
    def __getattr__(self, name):
        return lambda *a: None


def _calls(b, kind, x, bits, outs=None):
    """One pass through the four entry points of a quantizer family; every call's (name, args) and result."""
    rot = kind.startswith("rot_")
    q = kind[4:] if rot else kind
    quantizer = {"asym": b.QUANTIZER_ASYM, "sym": b.QUANTIZER_SYM, "fp8": b.QUANTIZER_FP8, "cmeta": None}[q]
    sfx = "" if q == "asym" else "_" + q
    n, t, h = x.shape
    g = 128
    width = () if q == "fp8" else (bits,)
    made = []

    def call(name, *args, out=None):
        made.append((name, (*args, out), getattr(b, name)(*args, out=out)))
        return made[-1][2]

    outs = outs or {}
    parts = []
    for j in range(n):
        if rot:
            parts.append(call("quantize_rot", x[j], g, bits, quantizer, out=outs.get("q")))
        else:
            parts.append(call("quantize" + sfx, x[j], g, *width, out=outs.get("q")))
        parts[-1] = tuple(None if p is None else p.clone() for p in parts[-1])
    arrays = [torch.stack(p) for p in zip(*parts) if p[0] is not None]
    c = call("dequant_reduce_requant" + sfx, *arrays, h, g, *(width * 2), out=outs.get("f"))
    if rot:
        call("dequantize_rot", c[0], c[1], c[2] if q == "asym" else None, h, g, bits, quantizer, out=outs.get("d"))
        name, extra = "allreduce_sim_rot", (bits, bits, quantizer)
    else:
        call("dequantize" + sfx, *c, h, g, *width, out=outs.get("d"))
        name, extra = "allreduce_sim" + sfx, width * 2
    made.append((name, (x, g, *extra, None, None), getattr(b, name)(x, g, *extra)))
    ws = torch.empty(b.allreduce_sim_workspace_bytes(n, t, h, g, bits, bits), dtype=torch.uint8, device="cuda")
    y = torch.empty(t, h, dtype=torch.float16, device="cuda")
    made.append((name, (x, g, *extra, y, ws), getattr(b, name)(x, g, *extra, out=y, workspace=ws)))
    assert made[-1][2] is y
    return made


def _flat(results):
    return [t for r in results for t in (r if isinstance(r, tuple) else (r,)) if t is not None]


@pytest.mark.gpu
@pytest.mark.parametrize("kind,bits", [(k, w) for k in KINDS for w in (4, 8) if w == 8 or not k.endswith("fp8")])
def test_native_calls_give_what_the_checked_path_gives(monkeypatch, kind, bits):
    from paper_2412_04964_amd import binding as b
    torch.manual_seed(1)
    x = torch.randn(3, 5, 1024, device="cuda").half()
    q = kind.replace("rot_", "")
    code = lambda w: torch.empty(5, 1024 * w // 8, dtype=torch.uint8, device="cuda")
    meta = lambda: torch.empty(5, 8, dtype=torch.int32 if q == "cmeta" else torch.float32, device="cuda")
    coded = lambda: (code(bits), *[meta() for _ in range(2 if q == "asym" else 1)])
    outs = {"q": coded(), "f": list(coded()), "d": torch.empty(5, 1024, dtype=torch.float16, device="cuda")}

    got = {}
    for given in (None, outs):
        made = _calls(b, kind, x, bits, given)
        native = b._calls()
        for name, args, _ in made:                        # the native module takes every one of these calls
            assert getattr(native, name)(*args) is not None, name
        got[given is None] = [t.clone() for t in _flat(r for _, _, r in made)]
        with monkeypatch.context() as m:
            m.setattr(b, "_native", Declines())
            want = _flat(r for _, _, r in _calls(b, kind, x, bits, given))
        assert len(want) == len(got[given is None])
        for g, w in zip(got[given is None], want):
            assert g.shape == w.shape and g.dtype == w.dtype and torch.equal(g, w)


@pytest.mark.gpu
def test_native_calls_leave_everything_else_to_the_checked_path():
    from paper_2412_04964_amd import binding as b
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Sub(torch.Tensor):
        pass

    x = torch.randn(4, 1024, device="cuda").half()
    q = b._calls().quantize
    assert q(x, 128, 4, None) is not None
    out = b.quantize(x, 128, 4)
    for args in [(x.float(), 128, 4, None), (x.cpu(), 128, 4, None), (x.t(), 128, 4, None), (x[0], 128, 4, None),
                 (x.as_subclass(Sub), 128, 4, None), (x, 96, 4, None), (x, 2048, 4, None), (x, 128, 5, None),
                 (x, 128.0, 4, None), (x, 128, True, None), (x, 1 << 40, 4, None), (x, 128, 4),
                 (x, 128, 4, out[:2]), (x, 128, 4, (out[0], out[1], out[2][:3])), (x, 128, 4, iter(out)),
                 (x, 128, 4, (out[1], out[0], out[2])), (None, 128, 4, None)]:
        assert q(*args) is None, args[1:]
    class Seen(TorchFunctionMode):
        def __torch_function__(self, fn, types, args=(), kwargs=None):
            return fn(*args, **(kwargs or {}))
    class Dispatched(TorchDispatchMode):
        def __torch_dispatch__(self, fn, types, args=(), kwargs=None):
            return fn(*args, **(kwargs or {}))
    for mode in (Seen, Dispatched):
        with mode():
            assert q(x, 128, 4, None) is None
            assert torch.equal(b.quantize(x, 128, 4)[0], out[0])

    def transformed(row):
        assert q(row, 128, 4, None) is None
        return row
    torch.func.vmap(transformed)(x[None])
    with torch.inference_mode():                          # an ordinary context: taken, same result
        assert torch.equal(q(x, 128, 4, None)[0], out[0])
    p = torch.nn.Parameter(x)
    assert not b.quantize(p, 128, 4)[1].requires_grad and torch.equal(q(p, 128, 4, None)[0], out[0])
    # refused by the library after the module's checks: the binding's error
    odd = torch.zeros(4 * 1024 + 1, dtype=torch.float16, device="cuda")[1:].view(4, 1024)
    with pytest.raises(b.FcError) as e:
        b.quantize(odd, 128, 4)
    assert e.value.code == -5


@pytest.mark.gpu
def test_native_calls_go_to_the_current_stream():
    from paper_2412_04964_amd import binding as b
    x = torch.randn(2, 64, 1024, device="cuda").half()
    want = b.allreduce_sim(x, 128, 4, 4)
    src, y = torch.zeros_like(x), torch.empty_like(want)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for _ in range(20):
            src.copy_(torch.zeros_like(x))                # ordered on s alone: each call sees the last copy of s
            torch.cuda._sleep(200000)
            src.copy_(x)
            assert b._calls().allreduce_sim(src, 128, 4, 4, y, None) is y
    s.synchronize()
    assert torch.equal(y, want)


@pytest.mark.gpu
def test_a_list_of_outputs_may_change_during_the_call():
    # Another thread runs while the library is called without the interpreter lock.  It exchanges the entries of a list
    # of outputs (always as a whole): the call must return the tensors that it wrote.
    from paper_2412_04964_amd import binding as b
    x = torch.randn(8, 1024, device="cuda").half()
    want = b.quantize(x, 128, 4)
    rot = b.quantize_rot(x, 128, 4, b.QUANTIZER_SYM)
    sets = [[torch.empty_like(t) for t in want] for _ in range(2)]
    shared, stop = list(sets[0]), threading.Event()

    def exchange():
        while not stop.is_set():
            shared[:] = sets[1]
            shared[:] = sets[0]

    thread, interval = threading.Thread(target=exchange), sys.getswitchinterval()
    sys.setswitchinterval(1e-6)
    thread.start()
    try:
        for i in range(300):
            for t in sets[0] + sets[1]:
                t.zero_()
            if i % 2:
                got, expected = b.quantize(x, 128, 4, out=shared), want
            else:
                got, expected = b.quantize_rot(x, 128, 4, b.QUANTIZER_SYM, out=shared)[:2], rot[:2]
            assert any(all(g is t for g, t in zip(got, s)) for s in sets), "tensors of two sets"
            assert all(torch.equal(g, w) for g, w in zip(got, expected)), "tensors that were not written"
    finally:
        stop.set()
        thread.join()
        sys.setswitchinterval(interval)


@pytest.mark.parametrize("why", ["missing", "other torch"])
def test_without_the_native_module_the_checked_path_takes_every_call(monkeypatch, why):
    import paper_2412_04964_amd
    from paper_2412_04964_amd import binding as b
    monkeypatch.setattr(b, "_native", None)
    if why == "missing":
        monkeypatch.delattr(paper_2412_04964_amd, "_fc_torch", raising=False)
        monkeypatch.setitem(sys.modules, "paper_2412_04964_amd._fc_torch", None)
    else:
        from paper_2412_04964_amd import _fc_torch
        monkeypatch.setattr(_fc_torch, "torch_version", "0")
    reached = []
    monkeypatch.setattr(b, "_dev", lambda t, dtype, what: t)
    monkeypatch.setattr(b, "_check", lambda rc, what: reached.append(what))
    monkeypatch.setattr(b, "_stream", lambda: 0)
    empty = torch.zeros(0, 256, dtype=torch.float16)      # a call that launches nothing
    with pytest.warns(RuntimeWarning, match="_fc_torch"):
        codes, scales, zeros = b.quantize(empty, 128, 4)
    with warnings.catch_warnings():
        warnings.simplefilter("error")                    # no second warning
        b.dequantize(codes, scales, zeros, 256, 128, 4)
    b.allreduce_sim(empty[None], 128, 4, 4)
    assert reached == ["fc_quantize", "fc_dequantize", "fc_allreduce_sim"]


def test_native_module_takes_no_cpu_tensor():
    from paper_2412_04964_amd import binding as b
    x = torch.zeros(4, 256, dtype=torch.float16)
    assert b._calls().quantize(x, 128, 4, None) is None
    assert b._calls().allreduce_sim(x[None], 128, 4, 4, None, None) is None
    with pytest.raises(TypeError):
        b.quantize(x, 128, 4)


@pytest.mark.gpu
@pytest.mark.parametrize("inference", [False, True])
def test_allocated_results_are_tensors_like_those_of_torch_empty(inference):
    # the native calls allocate without torch's dispatcher: type, place, layout, storage, autograd state and the allocator's
    # bookkeeping are those of torch.empty
    from paper_2412_04964_amd import binding as b
    x = torch.randn(3, 5, 1024, device="cuda").half()
    with torch.inference_mode(inference):
        for t in [*b.quantize(x[0], 128, 4), b.allreduce_sim(x, 128, 4, 8), b.quantize_cmeta(x[0][:0], 128, 8)[1]]:
            like = torch.empty(tuple(t.shape), dtype=t.dtype, device="cuda")
            assert type(t) is type(like) and t.device == like.device and t.stride() == like.stride()
            assert t.untyped_storage().nbytes() == like.untyped_storage().nbytes() and t.storage_offset() == 0
            assert t.requires_grad == like.requires_grad and t.is_inference() == like.is_inference()
            t.record_stream(torch.cuda.current_stream())
    # A count that only grows: memory that earlier tests left to Python's collector may be freed between the two readings.
    allocated = lambda: torch.cuda.memory_stats()["allocated_bytes.all.allocated"]
    before = allocated()
    kept = b._calls().quantize(x[0], 128, 8, None)
    after = allocated()
    for k in kept:
        torch.empty_like(k)
    assert after - before == allocated() - after >= sum(k.untyped_storage().nbytes() for k in kept) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["allreduce_sim", "allreduce_sim_sym", "allreduce_sim_fp8", "allreduce_sim_cmeta", "allreduce_sim_rot"])
@pytest.mark.parametrize("n,t,h,g", [(2, 3, 1024, 32), (1, 1, 2048, 1024), (3, 520, 4096, 2048), (8, 0, 1024, 128)])
def test_all_reduce_without_a_workspace_allocates_its_result(name, n, t, h, g):
    # the rotated call also a workspace; the result is the one with a workspace given
    from paper_2412_04964_amd import binding as b
    x = torch.randn(n, t, h, device="cuda").half()
    args = (g,) if name.endswith("fp8") else (g, 4, 8)
    need = b.allreduce_sim_workspace_bytes(n, t, h, g, *(args[1:] or (8, 8)))
    space = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    extra = (b.QUANTIZER_ASYM,) if name.endswith("rot") else ()
    want = getattr(b, name)(x, *args, *extra, workspace=space)
    allocated = lambda: torch.cuda.memory_stats()["allocated_bytes.all.allocated"]
    before = allocated()
    got = getattr(b._calls(), name)(x, *args, *extra, None, None)
    new = allocated() - before
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert (new > want.numel() * 2 + 511) == name.endswith("rot") or t == 0


@pytest.mark.gpu
def test_allocated_results_are_filled_where_torch_was_asked_to():
    # torch.use_deterministic_algorithms has torch.empty fill new memory.  The kernels overwrite every byte of it, so what shows
    # the fill is torch's own record of the operations that ran: one per result.
    from paper_2412_04964_amd import binding as b
    x = torch.randn(5, 1024, device="cuda").half()
    got = {}
    for fill in (False, True):
        torch.use_deterministic_algorithms(fill)
        try:
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU], acc_events=True) as record:
                got[fill] = b._calls().quantize(x, 128, 8, None)
        finally:
            torch.use_deterministic_algorithms(False)
        assert got[fill] is not None
        assert sum(e.count for e in record.key_averages() if e.key == "aten::fill_") == (3 if fill else 0)
    assert all(torch.equal(a, w) for a, w in zip(got[True], got[False]))
