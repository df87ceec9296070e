"""The native marshalling of the attention calls (csrc/marshal.cpp) against the Python code beside it: same outputs, same errors."""
import ctypes
import threading
import time

import pytest
import torch
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2407_12117_amd import binding as mb
from paper_2407_12117_amd import synth

pytestmark = pytest.mark.gpu


class Wrapped(torch.Tensor):
    """A subclass: the native code leaves it to Python."""


def _calls(q, k, v, g, scale, as_given, lse=None):
    o, lse = mb.memo_attn_fwd(q, k, v, scale, o=torch.empty_like(q) if as_given else None, lse=lse)
    grads = [torch.empty_like(q) for _ in range(3)] if as_given else [None] * 3
    ws = torch.empty(mb.memo_attn_bwd_workspace_bytes(q, scale), dtype=torch.uint8, device="cuda") if as_given else None
    out = (o, lse) + mb.memo_attn_bwd(q, k, v, o, lse, g, scale, *grads, workspace=ws)
    return out + mb.memo_attn_bwd_static(q, k, v, o, lse, g, scale, *(torch.empty_like(q) for _ in range(3)))


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 128)])
@pytest.mark.parametrize("as_given", [False, True])
@pytest.mark.parametrize("side_stream", [False, True])
def test_native_and_python_marshalling_agree(dtype, d, as_given, side_stream):
    scale = synth.default_scale(d)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(2, 75, 3, d, dtype, 5))
    torch.cuda.synchronize()
    taken = mb._marshal().attn_fwd(mb.lib().address["memo_attn_fwd"], mb._stream_ptr, q, k, v, scale, None, None, None)
    assert type(taken) is tuple                       # plain device tensors are taken
    assert mb._marshal().attn_fwd(mb.lib().address["memo_attn_fwd"], mb._stream_ptr, q.as_subclass(Wrapped), k, v, scale, None, None, None) is None
    with torch.cuda.stream(torch.cuda.Stream() if side_stream else torch.cuda.current_stream()):
        native = _calls(q, k, v, g, scale, as_given)
        plain = _calls(*(t.as_subclass(Wrapped) for t in (q, k, v, g)), scale, as_given)
    torch.cuda.synchronize()
    for x, y in zip(native, plain):
        assert x.shape == y.shape and x.stride() == y.stride() and x.dtype == y.dtype and torch.equal(x, y.as_subclass(torch.Tensor))


def test_errors_are_those_of_the_python_code():
    q = torch.zeros(1, 40, 2, 128, dtype=torch.bfloat16, device="cuda")
    lse, scale = torch.zeros(1, 2, 40, device="cuda"), 0.1
    for bad in (q[:, :32], q.float(), q.cpu(), q.transpose(1, 2).contiguous().transpose(1, 2)):
        with pytest.raises(ValueError, match="share shape|one device"):
            mb.memo_attn_fwd(q, bad, q, scale)
        with pytest.raises(ValueError, match="share shape|one device"):
            mb.memo_attn_bwd_static(q, q, q, q, lse, q, scale, q, bad, q)
    with pytest.raises(ValueError, match="lse must be"):
        mb.memo_attn_fwd(q, q, q, scale, o=torch.empty_like(q), lse=lse[:, :, :39])
    with pytest.raises(ValueError, match="unsupported dtype"):
        mb.memo_attn_fwd(*(q.half(),) * 3, scale)
    for f32_only, s in ((torch.zeros(1, 8, 1, 96, device="cuda"), scale), (q, -1.0)):
        with pytest.raises(mb.MemoError):
            mb.memo_attn_fwd(f32_only, f32_only, f32_only, s)
    with pytest.raises(mb.MemoError):                 # a workspace that is too small
        mb.memo_attn_bwd(q, q, q, q, lse, q, scale, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    with pytest.raises(AttributeError):
        mb.memo_attn_fwd(None, q, q, scale)


def test_buffers_that_are_too_small_are_refused_on_the_host():
    q = torch.zeros(1, 40, 2, 128, dtype=torch.bfloat16, device="cuda")
    lse, scale, out = torch.zeros(1, 2, 40, device="cuda"), 0.1, [torch.empty_like(q) for _ in range(3)]
    for bad, text in ((lse[:, :, :39], "lse must be"), (lse[:, :, :39].contiguous(), "lse must be"), (lse.bfloat16(), "lse must be"), (lse.cpu(), "one device")):
        for call in (lambda: mb.memo_attn_bwd(q, q, q, q, bad, q, scale), lambda: mb.memo_attn_bwd_static(q, q, q, q, bad, q, scale, *out)):
            with pytest.raises(ValueError, match=text):
                call()
    with pytest.raises(ValueError, match="one device"):
        mb.memo_attn_fwd(q, q, q, scale, lse=lse.cpu())
    need = mb.memo_attn_bwd_workspace_bytes(q, scale)
    few = torch.zeros(1, dtype=torch.uint8, device="cuda")
    for bad, text in ((few.expand(need), "workspace must be"), (torch.zeros(need, dtype=torch.uint8), "one device")):
        with pytest.raises(ValueError, match=text):
            mb.memo_attn_bwd(q, q, q, q, lse, q, scale, workspace=bad)


def test_buffers_of_other_forms_are_still_taken():
    # an lse without its shape, a longer one, a workspace that is a view, of another type or with gaps: enough memory in every case
    scale = synth.default_scale(64)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(1, 75, 2, 64, "f32", 6))
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    want = mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    need = mb.memo_attn_bwd_workspace_bytes(q, scale)
    longer = torch.cat([lse.flatten(), torch.full((7,), float("nan"), device="cuda")])
    room = torch.zeros(4 * need, dtype=torch.uint8, device="cuda")
    for some_lse, workspace in ((lse.view(2, 75), None), (lse.flatten(), room), (longer, room[256:]), (lse, room[::2]), (lse, room.view(torch.float32)),
                                (lse.cpu().pin_memory(), room.view(2, -1)), (lse, torch.zeros(need, dtype=torch.uint8, pin_memory=True))):
        for x, y in zip(mb.memo_attn_bwd(q, k, v, o, some_lse, g, scale, workspace=workspace), want):
            assert torch.equal(x, y)


def _native(q, k, v, g, scale):
    """What the native code alone makes of a forward and a backward: their outputs, or None where it leaves a call to Python."""
    at, native = mb.lib().address, mb._marshal()
    fwd = native.attn_fwd(at["memo_attn_fwd"], mb._stream_ptr, q, k, v, scale, None, None, None)
    o, lse = fwd if fwd is not None else (torch.empty_like(q), torch.empty(q.shape[0], q.shape[2], q.shape[1], device=q.device))
    return fwd, native.attn_bwd(at["memo_attn_bwd"], at["memo_attn_bwd_workspace_bytes"], mb._stream_ptr, q, k, v, o, lse, g, scale, None, None, None, None, None)


def _case(seed):
    return [t.cuda() for t in synth.attn_inputs(1, 75, 2, 64, "f32", seed)] + [synth.default_scale(64)]


def test_tensors_that_require_grad_and_inference_tensors_are_taken():
    q, k, v, g, scale = _case(8)
    want = [t for part in _native(q, k, v, g, scale) for t in part]
    for t in (q, k, v, g):
        t.requires_grad_()
    got = [t for part in _native(q, k, v, g, scale) for t in part]
    assert all(torch.equal(x, y) and not x.requires_grad for x, y in zip(got, want))
    with torch.inference_mode():
        q, k, v, g = (t.clone() for t in (q, k, v, g))
        got = [t for part in _native(q, k, v, g, scale) for t in part]
        assert all(torch.equal(x, y) and x.is_inference() for x, y in zip(got, want))


def test_modes_that_intercept_calls_see_the_python_code():
    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return func(*args, **(kwargs or {}))

    class Function(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(getattr(func, "__name__", str(func)))
            return func(*args, **(kwargs or {}))

    q, k, v, g, scale = _case(9)
    o, lse = mb.memo_attn_fwd(q, k, v, scale)
    want = (o, lse) + mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    for mode in (Dispatch, Function):
        seen = []
        with mode():
            assert _native(q, k, v, g, scale) == (None, None)
            seen.clear()
            o, lse = mb.memo_attn_fwd(q, k, v, scale)
            got = (o, lse) + mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
        assert sum("empty" in name for name in seen) >= 4        # the outputs are allocated where the mode sees it
        assert all(torch.equal(x, y) for x, y in zip(got, want))


def test_functorch_wrappers_are_left_to_python():
    q, k, v, g, scale = _case(10)

    def batched(x):
        left.append(_native(x, x, x, x, scale))
        with pytest.raises(RuntimeError):             # a wrapper has no memory of its own
            mb.memo_attn_fwd(x, x, x, scale)
        return x

    left = []
    torch.func.vmap(batched)(torch.stack((q, k)))
    torch.func.grad(lambda x: batched(x).sum())(q)
    assert left == [(None, None)] * 2


def test_calls_under_graph_capture():
    # outputs and workspace from the graph's pool; replayed on new inputs with eager work between
    q, k, v, g, scale = _case(11)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        mb.memo_attn_bwd(q, k, v, *mb.memo_attn_fwd(q, k, v, scale), g, scale)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, lse = mb.memo_attn_fwd(q, k, v, scale)
        got = (o, lse) + mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
    for seed in (12, 13, 14):
        for t, new in zip((q, k, v, g), _case(seed)):
            t.copy_(new)
        o, lse = mb.memo_attn_fwd(q, k, v, scale)
        want = (o, lse) + mb.memo_attn_bwd(q, k, v, o, lse, g, scale)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, want))


@pytest.mark.parametrize("handle", [None, 0, False, ctypes.c_void_p(None), ctypes.c_void_p(0), 1 << 64])
def test_stream_handles_that_ctypes_takes(handle):
    # the default stream in the forms in which a caller's own stream object may hold it
    class Stream:
        cuda_stream = handle

    scale = synth.default_scale(64)
    q, k, v, g = (t.cuda() for t in synth.attn_inputs(1, 75, 2, 64, "f32", 7))
    torch.cuda.synchronize()
    got = mb.memo_attn_fwd(q, k, v, scale, stream=Stream())
    got += mb.memo_attn_bwd(q, k, v, *got, g, scale, stream=Stream())
    got += mb.memo_attn_bwd_static(q, k, v, got[0], got[1], g, scale, *(torch.empty_like(q) for _ in range(3)), stream=Stream())
    torch.cuda.synchronize()
    want = mb.memo_attn_fwd(q, k, v, scale)
    grads = mb.memo_attn_bwd(q, k, v, *want, g, scale)
    for x, y in zip(got, want + grads + grads):
        assert torch.equal(x, y)


@pytest.mark.parametrize("backward", [False, True])
def test_other_threads_run_while_an_output_is_allocated(backward):
    # the allocator gives segments back to the device first, which waits for the work that is queued
    q = torch.zeros(64, 4096, 16, 128, dtype=torch.bfloat16, device="cuda")     # 1 GiB
    scale = synth.default_scale(128)
    o, lse = mb.memo_attn_fwd(q, q, q, scale)
    busy = torch.zeros(1, 131072, 4, 128, dtype=torch.bfloat16, device="cuda")
    busy_o, busy_lse = mb.memo_attn_fwd(busy, busy, busy, scale)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    outs = [torch.empty_like(q) for _ in range(2)]
    parts = [torch.empty(600 << 20, dtype=torch.uint8, device="cuda") for _ in range(2)]
    room = torch.cuda.memory_reserved() / torch.cuda.get_device_properties(0).total_memory
    del parts
    gaps, stop = [0.0], threading.Event()

    def watch():
        last = time.perf_counter()
        while not stop.is_set():
            time.sleep(0.001)
            now = time.perf_counter()
            gaps.append(now - last)
            last = now

    watcher = threading.Thread(target=watch)
    try:
        torch.cuda.set_per_process_memory_fraction(room)
        for _ in range(40):
            mb.memo_attn_fwd(busy, busy, busy, scale, o=busy_o, lse=busy_lse)
        watcher.start()
        time.sleep(0.02)
        begin = time.perf_counter()
        if backward:
            workspace = busy_o.view(torch.uint8).flatten()[:mb.memo_attn_bwd_workspace_bytes(q, scale)]
            mb.memo_attn_bwd(q, q, q, o, lse, q, scale, dk=outs[0], dv=outs[1], workspace=workspace)
        else:
            mb.memo_attn_fwd(q, q, q, scale, lse=lse)
        took = time.perf_counter() - begin
    finally:
        stop.set()
        if watcher.ident:
            watcher.join()
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    print(f"allocation took {took:.3f} s, the other thread's longest gap was {max(gaps):.3f} s", flush=True)
    assert took > 0.1                                 # it did wait
    assert max(gaps) < 0.3 * took
