"""The two forms of a swap copy (copy_swapped, csrc/memo_kernels.h) on both sides of the limits between them: blocks around 256 KiB, token rows of
1 to 64 KiB and others, blocks off 16 bytes; host memory that is not pinned; several pairs of streams at once; graph capture.  Bytes come back as they were."""
import pytest
import torch

from paper_2407_12117_amd import binding as mb

pytestmark = pytest.mark.gpu

KIB = 1024


def _act(rows, row_bytes, shift, seed):
    """[rows, row_bytes] bytes whose first one lies `shift` bytes from an aligned address."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    flat = torch.randint(0, 256, (rows * row_bytes + shift,), dtype=torch.uint8, device="cuda", generator=g)
    return flat[shift:].view(rows, row_bytes)


@pytest.mark.parametrize("rows,row_bytes,shift", [
    (63, 4 * KIB, 0), (64, 4 * KIB, 0), (64, 4 * KIB, 16), (64, 4 * KIB, 8), (65, 4 * KIB, 4),   # around the least size and the alignment
    (255, KIB, 0), (257, KIB, 0), (341, 3080, 0), (1000, 1001, 0), (1000, 1001, 1),              # token rows, and off 16 bytes
    (12345, 2560, 0), (1001, 1040, 16), (5, 64 * KIB, 0), (5, 64 * KIB + 16, 0),
    (4096, 128, 0), (4100, 128, 0), (33, 8 * KIB + 16, 0),                                       # rows of 4 KiB instead, or none
])
def test_bytes_come_back(rows, row_bytes, shift):
    print(f"[case] swap copy {rows} x {row_bytes} shift {shift}", flush=True)
    act = _act(rows, row_bytes, shift, 3)
    n = rows * row_bytes
    host = torch.full((n + 64 + shift,), 0xEE, dtype=torch.uint8, pin_memory=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    mb.memo_swap_out(act, 1.0, host[shift:], side)
    side.synchronize()
    assert torch.equal(host[shift:shift + n], act.cpu().view(-1)) and (host[shift + n:] == 0xEE).all() and (host[:shift] == 0xEE).all()
    back = torch.full((n + 2 * 64 + shift,), 0x5A, dtype=torch.uint8, device="cuda")
    side.wait_stream(torch.cuda.current_stream())
    mb.memo_swap_in(back[shift:shift + n].view(rows, row_bytes), 1.0, host[shift:], side)
    side.synchronize()
    assert torch.equal(back[shift:shift + n], act.view(-1)) and (back[shift + n:] == 0x5A).all() and (back[:shift] == 0x5A).all()


def test_host_memory_that_is_not_pinned():
    # the C entry points take it, as one block
    print("[case] swap copy, host memory not pinned", flush=True)
    rows, row_bytes = 100, 4 * KIB
    act = _act(rows, row_bytes, 0, 4)
    back = torch.zeros_like(act)
    host = torch.zeros(rows * row_bytes, dtype=torch.uint8)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for call, dev in ((mb.lib().memo_swap_out, act), (mb.lib().memo_swap_in, back)):
        assert call(dev.data_ptr(), rows, row_bytes, 1.0, host.data_ptr(), host.numel(), side.cuda_stream, None, None) == mb.MEMO_OK
        side.synchronize()
    assert torch.equal(host, act.cpu().view(-1)) and torch.equal(back, act)


def test_pairs_of_streams_at_once():
    pairs = [(_act(4096, 8 * KIB, 0, s), torch.zeros(4096 * 8 * KIB, dtype=torch.uint8, pin_memory=True), torch.cuda.Stream(), torch.cuda.Stream())
             for s in range(3)]
    backs = [torch.zeros_like(p[0]) for p in pairs]
    torch.cuda.synchronize()
    for _ in range(2):
        for (act, host, out, inn), back in zip(pairs, backs):
            done = torch.cuda.Event()
            mb.memo_swap_out(act, 1.0, host, out, done_event=done)
            mb.memo_swap_in(back, 1.0, host, inn, wait_event=done)
    torch.cuda.synchronize()
    for (act, host, _, _), back in zip(pairs, backs):
        assert torch.equal(back, act) and torch.equal(host, act.cpu().view(-1))


@pytest.mark.parametrize("rows,row_bytes", [(16, 4 * KIB), (300, 4 * KIB), (1000, 1001)])
def test_graph_capture(rows, row_bytes):
    act = torch.zeros((rows, row_bytes), dtype=torch.uint8, device="cuda")
    back = torch.zeros_like(act)
    host = torch.zeros(rows * row_bytes, dtype=torch.uint8, pin_memory=True)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        here = torch.cuda.current_stream()
        mb.memo_swap_out(act, 1.0, host, here)
        mb.memo_swap_in(back, 1.0, host, here)
    for seed in range(4):
        act.copy_(_act(rows, row_bytes, 0, seed))
        back.fill_(0x5A)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(back, act) and torch.equal(host, act.cpu().view(-1))
