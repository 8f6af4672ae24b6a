"""The native marshalling of calls answers as the Python marshalling does.

Every entry point is called twice on the same inputs: through the native module, and with
the module answering NotImplemented, which leaves the call to the Python code.  Outputs,
states, cached rows and bookkeeping have to be equal bit for bit, and a refusal has to be
the same exception, since both marshal into the same C call."""
import numpy as np
import pytest
import torch

import paper_2607_02805_amd as bd


class _Counting:
    """The native module, counting the calls that it takes."""

    def __init__(self, real):
        self.real, self.taken = real, 0

    def __getattr__(self, name):
        f = getattr(self.real, name)

        def run(*a):
            got = f(*a)
            self.taken += got is not NotImplemented
            return got
        return run


class _Absent:
    def __getattr__(self, name):
        return lambda *a: NotImplemented


B, L, H, G, N, NS = 2, 5, 4, 2, 32, 4


def _inputs(dtype, dev):
    g = torch.Generator().manual_seed(7)

    def r(*s):
        return torch.randn(*s, generator=g)
    ch = bd.conv_channels(H, G, N)
    base = r(B, L, H * 64 + 2 * G * N + H).mul(0.3).to(dtype).to(dev)
    x = base[..., :H * 64].unflatten(2, (H, 64))                       # slices of one projection
    Bm = base[..., H * 64:H * 64 + G * N].unflatten(2, (G, N))
    Cm = base[..., H * 64 + G * N:H * 64 + 2 * G * N].unflatten(2, (G, N))
    dt = (r(B, L, H).abs() * 0.1).to(dtype).to(dev)
    v = {"x": x, "dt": dt, "B": Bm, "C": Cm, "A": -r(H).abs().to(dev) - 0.1, "D": r(H).to(dev),
         "Dr": r(H).to(dev), "w": (r(ch, 4) * 0.3).to(dev), "b": r(ch).to(dev) * 0.1,
         "z": r(B, L, H * 64).to(dtype).to(dev), "nw": r(H * 64).to(dev)}
    v["h0"], v["c0"] = r(*bd.pool_shape(NS, H, N)).to(dev), r(NS, 3, ch).to(dev)
    return v


def _calls(v, h, c, nc, nb, slots):
    act = (v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"])
    raw = (v["x"], v["dt"], v["B"], v["C"])
    book = (nc, nb)
    shape = (B, L, H, 64)
    yy = torch.empty(shape, device=h.device)
    s = torch.cuda.current_stream() if h.is_cuda else None
    kw = dict(slot_idx=slots)
    return {
        "step": lambda: bd.scan_block_step(*act, v["Dr"], h, **kw),
        "step_y": lambda: bd.scan_block_step(*act, v["Dr"], h, y=yy, stream=s, **kw),
        "sep": lambda: bd.scan_block_step_sep(act, act[:5] + (v["Dr"],), h, **kw),
        "commit": lambda: bd.commit_boundary(*act, v["Dr"], h, *book, **kw),
        "commit_y": lambda: bd.commit_boundary(*act, v["Dr"], h, *book, y_clean=True, **kw),
        "commit_step": lambda: bd.commit_step(raw, raw, v["A"], v["D"], v["Dr"], h, *book,
                                              y_clean=True, **kw),
        "conv_step": lambda: bd.conv_block_step(*act, v["Dr"], v["w"], v["b"], c, h, **kw),
        "conv_commit": lambda: bd.conv_commit_boundary(*act, v["Dr"], v["w"], v["b"], c, h, *book, **kw),
        "window": lambda: bd.scan_full_window(*act, v["Dr"]),
        "prefill": lambda: bd.prefill(*act, h, *book, blocks_in_prefix=1, y_fwd=True, **kw),
        "prefill_noalloc": lambda: bd.prefill_noalloc(*act, h, *book, blocks_in_prefix=1, y_fwd=yy, **kw),
        "norm": lambda: bd.gated_rmsnorm(yy.fill_(0.5), v["z"], v["nw"], 1e-5, 2),
        # refused by the C ABI: a repeated or missing slot, books that do not match
        "bad_slot": lambda: bd.commit_boundary(*act, v["Dr"], h, *book, slot_idx=np.array([1, 1], np.int32)),
        "far_slot": lambda: bd.scan_block_step(*act, v["Dr"], h, slot_idx=np.array([0, NS], np.int32)),
        "bad_book": lambda: bd.commit_boundary(*act, v["Dr"], h, *book, expected_block_index=3, **kw),
        # left to the Python code, which converts or refuses
        "list_slots": lambda: bd.scan_block_step(*act, v["Dr"], h, slot_idx=[3, 0]),
        "short_y": lambda: bd.scan_block_step(*act, v["Dr"], h, y=yy[:, :-1], **kw),
        "flat_pool": lambda: bd.scan_block_step(*act, v["Dr"], h.flatten(2), **kw),
        "half_x": lambda: bd.scan_block_step(v["x"].half(), *act[1:], v["Dr"], h, **kw),
        "cut_sep": lambda: bd.scan_block_step_sep(act[:5], act + act[:1], h, **kw),
        "cpu_A": lambda: bd.scan_block_step(*act[:2], v["A"].cpu(), *act[3:], v["Dr"], h, **kw),
    }


PLAIN = ("step", "step_y", "sep", "commit", "commit_y", "commit_step", "conv_step", "conv_commit",
         "window", "prefill", "prefill_noalloc", "norm", "bad_slot", "far_slot", "bad_book")
OTHER = ("list_slots", "short_y", "flat_pool", "half_x", "cut_sep", "cpu_A")


def _run(monkeypatch, native, name, dtype, slots, dev):
    monkeypatch.setattr(bd, "_marshal", native)
    v = _inputs(dtype, dev)
    h, c = v["h0"].clone(), v["c0"].clone()
    nc, nb = np.zeros(NS, np.int64), np.zeros(NS, np.int64)
    err = out = None
    try:
        out = _calls(v, h, c, nc, nb, slots)[name]()
    except Exception as e:                                # compared between the two sides
        err = (type(e), str(e))
    if h.is_cuda:
        torch.cuda.synchronize()
    outs = [t for t in (out if isinstance(out, tuple) else (out,)) if t is not None]
    return err, [t.cpu() for t in outs + [h, c]] + [torch.from_numpy(nc), torch.from_numpy(nb)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("slotted", [False, True])
@pytest.mark.parametrize("name", PLAIN + OTHER)
def test_native_and_python_marshalling_agree(monkeypatch, name, slotted, dtype):
    slots = np.array([3, 1], np.int32) if slotted else None
    native = _Counting(bd._native())
    err, got = _run(monkeypatch, native, name, dtype, slots, "cuda")
    err2, want = _run(monkeypatch, _Absent(), name, dtype, slots, "cuda")
    assert native.taken == (name in PLAIN)
    assert err == err2 and len(got) == len(want)
    for a, b in zip(got, want):
        assert a.dtype == b.dtype and torch.equal(a, b)


@pytest.mark.parametrize("name", [n for n in PLAIN + OTHER if n != "step_y"])
def test_tensors_off_the_gpu_are_refused_as_before(monkeypatch, name):
    native = _Counting(bd._native())
    err, _ = _run(monkeypatch, native, name, torch.float32, None, "cpu")
    err2, _ = _run(monkeypatch, _Absent(), name, torch.float32, None, "cpu")
    assert native.taken == 0 and err is not None and err == err2


@pytest.mark.gpu
def test_intercepted_calls_are_left_to_python():
    """Tensor subclasses and modes see the operations that the Python code makes: calls that
    the native module takes are left to Python under a mode, or with a subclass among them."""
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Functions(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    class Sub(torch.Tensor):
        pass

    n = bd._native()
    v = _inputs(torch.float32, "cuda")
    act = [v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"], v["Dr"], v["h0"], None,
           np.array([3, 1], np.int32), None]
    y = torch.ones(B, L, H, 64, device="cuda")
    norm = [y, v["z"], v["nw"], 1e-5, 1, None, None]
    for f, args, tensors in ((n.scan_block_step, act, (0, 1, 2, 3, 4, 5, 6, 7)), (n.gated_rmsnorm, norm, (0, 1, 2))):
        assert torch.is_tensor(f(*args))
        for mode in (Functions, Dispatch):
            with mode():
                assert f(*args) is NotImplemented
        with torch.device("meta"):
            assert f(*args) is NotImplemented
        for i in tensors:
            sub = list(args)
            sub[i] = args[i].as_subclass(Sub)
            assert f(*sub) is NotImplemented
        assert torch.is_tensor(f(*args))
        assert f(*args[:-1]) is NotImplemented
    torch.cuda.synchronize()


def test_native_module_missing_is_loud(monkeypatch, tmp_path):
    monkeypatch.setattr(bd, "_marshal", None)
    monkeypatch.setattr(bd, "BIND_PATH", str(tmp_path / "_bind.so"))
    with pytest.raises(RuntimeError, match="missing"):
        bd._native()
