"""Validations captured in a graph beside the program's own work on another stream."""
import pytest
import torch

from gpu_util import guard_mod, need_gpu
from synth import make_queries, make_table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("still_copying", [False, True])
def test_capture_beside_a_stream_that_copied_the_byte_index(still_copying):
    """A bulk validation queues the copy of the byte index on its stream. A stream that is being captured
    can neither wait for it nor ask whether it is done, and has no need to: its validations take the
    general path."""
    need_gpu()
    g = guard_mod()
    R, n, big = 20_000, (1 << 20) + 5, 20_000 << 10
    tb = make_table(R, 64, 3)
    rt = g.RangeTable(R)
    rt.insert_many(tb.base, tb.size, tb.kind)
    q = make_queries(tb, n, 4).cuda()
    bulk = q.repeat(big // n + 1, 1).contiguous()
    verdict = torch.empty(bulk.shape[0], dtype=torch.uint8, device="cuda")
    owner = torch.empty(bulk.shape[0], dtype=torch.int32, device="cuda")
    out = [(torch.zeros(m, dtype=torch.uint8, device="cuda"), torch.zeros(m, dtype=torch.int32, device="cuda"))
           for m in (1000, n, n)]
    want = [torch.empty_like(x) for x in out[1]]
    own, captured = torch.cuda.Stream(), torch.cuda.Stream()
    g.agile_validate_ptrs(rt.handle, q, n, *want, own)
    torch.cuda.synchronize()
    with torch.cuda.stream(captured):
        g.agile_validate_ptrs(rt.handle, q, 1000, *out[0])  # the table is known to be there
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    if still_copying:
        with torch.cuda.stream(own):
            torch.cuda._sleep(400_000_000)  # the copy waits behind this
    g.agile_validate_ptrs(rt.handle, bulk, bulk.shape[0], verdict, owner, own)
    if not still_copying:
        torch.cuda.synchronize()
    with torch.cuda.stream(captured):
        graph.capture_begin()
        g.agile_validate_ptrs(rt.handle, q, 1000, *out[0])
        g.agile_validate_ptrs(rt.handle, q, n, *out[1])
        graph.capture_end()
    assert own.query() != still_copying
    g.agile_validate_ptrs(rt.handle, q, n, *out[2])  # a stream that is not captured waits for it
    for rep in range(4):
        for x in out[0] + out[1]:
            x.fill_(77)
        graph.replay()
        torch.cuda.synchronize()
        for (v, o), m in zip(out, (1000, n, n)):
            assert torch.equal(v, want[0][:m]) and torch.equal(o, want[1][:m]), rep
        g.agile_validate_ptrs(rt.handle, q, n, *out[2])
    for k in range(0, big, n):
        m = min(n, bulk.shape[0] - k)
        assert torch.equal(verdict[k:k + m], want[0][:m]) and torch.equal(owner[k:k + m], want[1][:m]), k
    rt.close()
