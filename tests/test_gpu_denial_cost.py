"""Denied accesses are no more expensive than allowed ones by much: a client that aims its indices
outside its allocations must not slow down the launch that it shares the chip with. Each case times a
call with denials against the same call without any, on the same GPU and in turn, with a bound well
above what a launch needs for the exact path and well below what waiting for one memory place costs,
and checks the log's count and first record over all the calls."""
import numpy as np
import pytest
import torch

from gpu_util import guard_mod, need_gpu

pytestmark = pytest.mark.gpu


def _times(calls, rounds=7):
    """Least milliseconds of each of `calls`, taken in turn."""
    best = [float("inf")] * len(calls)
    for r in range(rounds + 1):
        for k, call in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                call()
            b.record()
            b.synchronize()
            if r:
                best[k] = min(best[k], a.elapsed_time(b) / 3)
    return best


def _indices(n, rows, part, gen):
    """Uniform rows, and the same with `part` of them `rows + 3`: past the table."""
    good = torch.randint(0, rows, (n,), generator=gen, device="cuda")
    bad = torch.rand(n, generator=gen, device="cuda") < part
    bad[n // 3] = True
    return good, torch.where(bad, rows + 3, good), int(bad.sum()), int(bad.nonzero()[0])


@pytest.mark.parametrize("n,D,rows,part", [(1 << 24, 1, 1 << 26, 0.01), (1 << 24, 1, 1 << 26, 1.0),
                                           (1 << 20, 3, 1 << 24, 0.3), (1 << 24, 1, 1 << 20, 0.3)])
def test_denied_rows_of_a_gather_fold_without_waiting_for_each_other(n, D, rows, part):
    need_gpu()
    g = guard_mod()
    gen = torch.Generator(device="cuda").manual_seed(n + D)
    table = torch.rand(rows, D, generator=gen, device="cuda")
    out = torch.empty(n, D, device="cuda")
    good, mixed, nbad, first = _indices(n, rows, part, gen)
    rt = g.RangeTable(16)
    for t in (table, out, good, mixed):
        rt.insert_tensor(t)
    runs = [0]

    def denied():
        runs[0] += 1
        g.agile_guarded_gather(rt.handle, out, table, 4 * D, mixed, n)

    t_ok, t_bad = _times([lambda: g.agile_guarded_gather(rt.handle, out, table, 4 * D, good, n), denied])
    denied()
    assert torch.equal(out, torch.where((mixed < rows)[:, None], table[mixed.clamp(max=rows - 1)], 0.0))
    rc, f = rt.fault_log(clear=True)
    assert f["count"] == runs[0] * nbad * D and f["first_elem"] == first * D and f["first_operand"] == 1
    assert t_bad < 2.0 * t_ok, (t_ok, t_bad)
    rt.close()


@pytest.mark.parametrize("n,D,rows,part,bound", [(50_000, 256, 1 << 16, 0.3, 4.0), (50_000, 64, 1 << 18, 1.0, 6.0),
                                                 (1 << 20, 1, 1 << 24, 0.01, 2.6)])
def test_denied_rows_of_a_batched_gather_are_shared_by_their_lanes(n, D, rows, part, bound):
    """A row outside the table is zeroed by as many lanes as would have copied it, and its denials reach the
    request's record once per workgroup."""
    need_gpu()
    g = guard_mod()
    gen = torch.Generator(device="cuda").manual_seed(n + D)
    table = torch.rand(rows, D, generator=gen, device="cuda")
    out = torch.empty(n, D, device="cuda")
    good, mixed, nbad, first = _indices(n, rows, part, gen)
    rt = g.RangeTable(16)
    for t in (table, out, good, mixed):
        rt.insert_tensor(t)
    cs = g.agile_clients_create([rt])
    ptrs = torch.zeros(1, 2, dtype=torch.int64, device="cuda")
    verdict = torch.zeros(1, dtype=torch.uint8, device="cuda")
    owner = torch.zeros(1, dtype=torch.int32, device="cuda")
    result = torch.zeros(72, dtype=torch.uint8, device="cuda")

    def call(idx):
        q = np.zeros(1, dtype=g.REQUEST_DTYPE)
        q[0]["gather_out"], q[0]["gather_table"] = out.data_ptr(), table.data_ptr()
        q[0]["gather_idx"], q[0]["gather_n"], q[0]["gather_row_bytes"] = idx.data_ptr(), n, 4 * D
        return lambda: g.agile_batch_run(cs, q, ptrs, 0, verdict, owner, result)

    t_ok, t_bad = _times([call(good), call(mixed)])
    call(mixed)()
    assert torch.equal(out, torch.where((mixed < rows)[:, None], table[mixed.clamp(max=rows - 1)], 0.0))
    r = g.batch_results(result, 1)[0]
    assert r["done"] == 1 and r["count"] == nbad * D and r["first_elem"] == first * D
    assert t_bad < bound * t_ok, (t_ok, t_bad)
    g.agile_clients_destroy(cs)
    rt.close()


@pytest.mark.parametrize("n,D,part", [(33_000, 16, 1.0), (262_144, 1, 0.3)])
def test_denied_rows_of_a_scatter_add_take_a_group_of_lanes_each(n, D, part):
    """Rows aimed outside the destination, in calls that add chunk by chunk: as many at a time as
    allowed rows, not one per wave. Values of a power of two: every sum is exact."""
    need_gpu()
    g = guard_mod()
    rows = 1 << 16
    gen = torch.Generator(device="cuda").manual_seed(n + D)
    good, mixed, nbad, first = _indices(n, rows, part, gen)
    dst, src = torch.zeros(rows, D, device="cuda"), torch.full((n, D), 0.25, device="cuda")
    rt = g.RangeTable(16)
    for t in (dst, src, good, mixed):
        rt.insert_tensor(t)
    calls = [lambda i=i: g.agile_guarded_scatter(rt.handle, dst, 4 * D, i, src, n, 0, g.SCATTER_ADD)
             for i in (good, mixed)]
    t_ok, t_bad = _times(calls)
    rt.fault_log(clear=True)
    dst.zero_()
    calls[1]()
    want = torch.bincount(mixed[mixed < rows], minlength=rows).float() * 0.25
    assert torch.equal(dst, want[:, None].expand(rows, D))
    rc, f = rt.fault_log(clear=True)
    assert f["count"] == nbad * D and f["first_elem"] == first * D and f["first_operand"] == 2
    assert t_bad < 2.0 * t_ok, (t_ok, t_bad)
    rt.close()


@pytest.mark.parametrize("op", ["gather", "scatter"])
@pytest.mark.parametrize("n,D,rows,part", [(131_072, 256, 1 << 16, 0.1), (131_072, 256, 1 << 16, 1.0),
                                           (300_000, 256, 1 << 16, 0.1)])
def test_rows_outside_their_allocation_need_no_look_at_each_element(n, D, rows, part, op):
    need_gpu()
    g = guard_mod()
    gen = torch.Generator(device="cuda").manual_seed(n + D)
    table = torch.rand(rows, D, generator=gen, device="cuda")
    flat = torch.rand(n, D, generator=gen, device="cuda")
    good, mixed, nbad, first = _indices(n, rows, part, gen)
    rt = g.RangeTable(16)
    for t in (table, flat, good, mixed):
        rt.insert_tensor(t)
    if op == "gather":
        calls = [lambda i=i: g.agile_guarded_gather(rt.handle, flat, table, 4 * D, i, n) for i in (good, mixed)]
    else:
        calls = [lambda i=i: g.agile_guarded_scatter(rt.handle, table, 4 * D, i, flat, n) for i in (good, mixed)]
    t_ok, t_bad = _times(calls)
    rt.fault_log(clear=True)
    before = table.clone()
    calls[1]()
    if op == "gather":
        assert torch.equal(flat, torch.where((mixed < rows)[:, None], table[mixed.clamp(max=rows - 1)], 0.0))
    else:  # rows that no index names keep their values
        untouched = torch.bincount(mixed[mixed < rows], minlength=rows) == 0
        assert torch.equal(table[untouched], before[untouched])
    rc, f = rt.fault_log(clear=True)
    assert f["count"] == nbad * D and f["first_elem"] == first * D
    assert f["first_operand"] == (1 if op == "gather" else 2)
    assert t_bad < 1.4 * t_ok, (t_ok, t_bad)
    rt.close()
