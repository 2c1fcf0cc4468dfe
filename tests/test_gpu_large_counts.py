"""Calls that need more threads than one grid holds (2^32): their kernels loop over the rest. Nothing of
these sizes goes through the oracle: torch answers the same question in pieces."""
import pytest
import torch

from gpu_util import guard_mod, need_gpu

pytestmark = pytest.mark.gpu

PIECE = 1 << 27


@pytest.fixture(autouse=True)
def memory():
    need_gpu()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 180 GiB of device memory")
    yield
    torch.cuda.empty_cache()


def test_gather_of_2_31_rows_of_twelve_bytes():
    """Two threads a row, from an allocation of more than 32 MiB: 2^32 threads and some."""
    g = guard_mod()
    rows, n = 4_000_000, (1 << 31) + 77
    gen = torch.Generator(device="cuda").manual_seed(5)
    table = torch.rand(rows, 3, generator=gen, device="cuda")
    idx = torch.randint(0, rows, (n,), generator=gen, device="cuda")
    idx[-3] = rows + 2
    out = torch.empty(n, 3, device="cuda")
    rt = g.RangeTable(8)
    for t in (table, idx, out):
        rt.insert_tensor(t)
    g.agile_guarded_gather(rt.handle, out, table, 12, idx, n)
    for k in range(0, n, PIECE):
        i = idx[k:k + PIECE]
        want = torch.where((i < rows)[:, None], table[i.clamp(max=rows - 1)], 0.0)
        assert torch.equal(out[k:k + PIECE], want), k
    rc, f = rt.fault_log(clear=True)
    assert f["count"] == 3 and f["first_elem"] == 3 * (n - 3)
    rt.close()


def test_copy_of_64_gib():
    """A 16-byte vector a thread: 2^32 threads and some."""
    g = guard_mod()
    n = (64 << 30) + 53
    src = torch.empty((n + 7) // 8, dtype=torch.int64, device="cuda")
    for k in range(0, src.numel(), PIECE):
        m = min(PIECE, src.numel() - k)
        src[k:k + m] = torch.arange(k, k + m, device="cuda") * 0x9E3779B97F4A7C1
    dst = torch.zeros_like(src)
    rt = g.RangeTable(8)
    for t in (src, dst):
        rt.insert_tensor(t)
    g.agile_guarded_copy(rt.handle, dst, src, n)
    full = n // 8
    for k in range(0, full, PIECE):
        m = min(PIECE, full - k)
        assert torch.equal(dst[k:k + m], src[k:k + m]), k
    tail = dst[full:].view(torch.uint8)
    assert torch.equal(tail[:n - 8 * full], src[full:].view(torch.uint8)[:n - 8 * full])
    assert not tail[n - 8 * full:].any()
    rc, f = rt.fault_log()
    assert f["count"] == 0
    rt.close()
