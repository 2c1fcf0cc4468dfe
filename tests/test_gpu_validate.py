"""Batched pointer validation on the GPU against the oracle: bit-exact verdicts and owners."""
import os
import random

import numpy as np
import pytest
import torch

from gpu_util import Twin, need_gpu
from synth import make_table, make_queries
from oracle import U64_MAX

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(__file__), "golden")


def run_validate(tw, q_u64):
    """q_u64: numpy uint64 [n, 2] -> device verdicts/owners as numpy."""
    n = q_u64.shape[0]
    q = torch.from_numpy(q_u64.view(np.int64).copy()).cuda()
    v = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    o = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    tw.g.agile_validate_ptrs(tw.h, q, n, v, o)
    torch.cuda.synchronize()
    return v.cpu().numpy(), o.cpu().numpy()


def assert_same(tw, q_u64, what=""):
    v, o = run_validate(tw, q_u64)
    ev, eo = tw.ot.verdict_many(q_u64[:, 0], q_u64[:, 1])
    bad = np.flatnonzero((v != ev) | (o != eo))
    assert bad.size == 0, (what, bad.size, [(hex(int(q_u64[k, 0])), int(q_u64[k, 1]), int(v[k]),
                                            int(o[k]), int(ev[k]), int(eo[k])) for k in bad[:5]])
    return ev


def test_table1_fixture():
    need_gpu()
    tw = Twin(64)
    qs, exp = [], []
    for line in open(os.path.join(GOLDEN, "table1_layout.txt")):
        tok = line.split("#")[0].split()
        if not tok:
            continue
        a = [int(x, 0) for x in tok[1:]]
        if tok[0] == "insert":
            tw.insert(a[0], a[1], a[2])
        elif tok[0] == "remove":
            q = np.array(qs, dtype=np.uint64)
            v, o = run_validate(tw, q)
            assert [(int(x), int(y)) for x, y in zip(v, o)] == exp
            qs, exp = [], []
            tw.remove(a[0])
        else:
            qs.append([a[0], a[1]])
            exp.append((a[2], a[3]))
    v, o = run_validate(tw, np.array(qs, dtype=np.uint64))
    assert [(int(x), int(y)) for x, y in zip(v, o)] == exp
    tw.close()


def test_small_guard_config_1e6_queries():
    """64-range table (48 USER log-uniform 256 B-1 MiB, 16 protected 4-64 KiB), 10^6 queries."""
    need_gpu()
    tb = make_table(64, 16, 0)
    tw = Twin(64)
    tw.insert_table(tb)
    q = make_queries(tb, 1_000_000, 0).numpy().view(np.uint64)
    ev = assert_same(tw, q, "c0")
    counts = np.bincount(ev, minlength=4)
    assert counts.min() > 0
    tw.close()


def _boundary_queries(ot, rng):
    qs = []
    ents = ot.entries()
    for b, e, _, _ in ents:
        for a in (b - 2, b - 1, b, b + 1, e - 2, e - 1, e, e + 1):
            if 0 <= a <= U64_MAX:
                for ln in (0, 1, 2, 3, 7, 4096, 1 << 40, U64_MAX):
                    qs.append([a, ln])
    for _ in range(200):
        qs.append([rng.getrandbits(64), rng.choice([0, 1, 5, U64_MAX])])
    qs += [[0, 0], [U64_MAX, 1], [U64_MAX, U64_MAX]]
    return np.array(qs, dtype=np.uint64)


@pytest.mark.parametrize("seed", range(8))
def test_exhaustive_boundaries_random_tables(seed, monkeypatch):
    """Byte-granular bases (uncompressed splitters), adjacency, kinds, top of address space."""
    need_gpu()
    monkeypatch.setenv("AGILE_WIDE_RECORDS", "1" if seed % 2 else "0")
    rng = random.Random(seed)
    tw = Twin(512)
    pos = rng.choice([0, 1 << 40, U64_MAX - (1 << 20)])
    for _ in range(rng.randrange(1, 300)):
        pos += rng.choice([0, 0, 1, 3, rng.randrange(0, 5000)])
        size = rng.choice([1, 2, 7, 64, rng.randrange(1, 9000)])
        if pos + size > U64_MAX:
            break
        tw.insert(pos, size, rng.choice([0, 0, 0, 1, 2]))
        pos += size
    assert_same(tw, _boundary_queries(tw.ot, rng), f"seed {seed}")
    # remove a third of the ranges: freed ranges become holes (lazy re-upload)
    ids = [e[3] for e in tw.ot.entries()]
    for rid in ids[::3]:
        tw.remove(rid)
    assert_same(tw, _boundary_queries(tw.ot, rng), f"seed {seed} after removal")
    tw.close()


def test_empty_table_and_zero_queries():
    need_gpu()
    tw = Twin(8)
    q = np.array([[0, 0], [12345, 1], [U64_MAX, U64_MAX]], dtype=np.uint64)
    v, o = run_validate(tw, q)
    assert (v == 3).all() and (o == -1).all()
    tw.g.agile_validate_ptrs(tw.h, 0, 0, 0, 0)   # n == 0 is a no-op
    tw.insert(100, 10, 0)
    assert_same(tw, q, "one entry")
    tw.close()


@pytest.mark.parametrize("budget", ["1024", "4096"])
def test_two_level_search_small_lds_budget(budget, monkeypatch):
    """Tables larger than the LDS budget search their last levels in global memory."""
    need_gpu()
    monkeypatch.setenv("AGILE_LDS_BUDGET", budget)
    tb = make_table(4096, 512, 11)
    tw = Twin(4096)
    tw.insert_table(tb)
    q = make_queries(tb, 300_001, 11).numpy().view(np.uint64)
    assert_same(tw, q, f"budget {budget}")
    tw.close()


@pytest.mark.parametrize("lift", ["2", "4", "6", "8"])
@pytest.mark.parametrize("n_ranges", [64, 4096])
def test_every_unrolled_search_depth(n_ranges, lift, monkeypatch):
    """The packed-record search is unrolled for 2, 4, 6 and 8 lifting levels and a table picks
    the depth its radix runs need; AGILE_MIN_LIFT raises the depth (deeper is still exact: the
    staged splitters are followed by sentinels), so each variant runs against the oracle."""
    need_gpu()
    monkeypatch.setenv("AGILE_MIN_LIFT", lift)
    tb = make_table(n_ranges, n_ranges // 8, 20 + int(lift))
    tw = Twin(n_ranges)
    tw.insert_table(tb)
    q = make_queries(tb, 200_003, 20 + int(lift)).numpy().view(np.uint64)
    assert_same(tw, q, f"{n_ranges} ranges, lift {lift}")
    tw.close()


@pytest.mark.parametrize("wide", ["0", "1"])
def test_large_table_ragged_queries(wide, monkeypatch):
    """65,536 ranges (8,192 protected) and a query count that is not a multiple of any tile,
    with the packed 16-byte bucket records and with the general 32-byte ones."""
    need_gpu()
    monkeypatch.setenv("AGILE_WIDE_RECORDS", wide)
    tb = make_table(65536, 8192, 1)
    tw = Twin(65536)
    tw.insert_table(tb)
    q = make_queries(tb, (1 << 22) + 77, 1).numpy().view(np.uint64)
    ev = assert_same(tw, q, "65536 ranges")
    assert np.bincount(ev, minlength=4).min() > 0
    tw.close()


def test_insert_remove_interleaved_with_validation():
    need_gpu()
    tw = Twin(256)
    rng = random.Random(5)
    live = []
    for step in range(40):
        if live and rng.random() < 0.3:
            tw.remove(live.pop(rng.randrange(len(live))))
        else:
            base = rng.randrange(0, 1 << 20) * 4096
            try:
                live.append(tw.insert(base, rng.randrange(1, 1 << 16), rng.choice([0, 1, 2])))
            except tw.g.AgileError as e:
                assert e.code == tw.g.AGILE_EOVERLAP      # both tables rejected it
        q = _boundary_queries(tw.ot, rng)
        assert_same(tw, q, f"step {step}")
    tw.close()


@pytest.mark.parametrize("n_ranges,far,lift", [(64, False, None), (1000, False, "8"),
                                               (1100, True, None), (8192, False, None),
                                               (8192, False, "6"), (9000, True, None),
                                               (13000, False, None), (15100, False, None)])
def test_bulk_queries_with_records_in_lds(n_ranges, far, lift, monkeypatch):
    """From 786,432 queries on, tables whose packed records fit the LDS behind the index are checked from
    there, with as many workgroups as fit or, for more than 2^24 queries, one per CU: small and large
    tables on either side of that, with 32-bit and 64-bit splitter keys (a far range makes the span too
    wide), pointer and DMA queries, a ragged count."""
    need_gpu()
    if lift:
        monkeypatch.setenv("AGILE_MIN_LIFT", lift)
    tb = make_table(n_ranges, n_ranges // 8, n_ranges)
    tw = Twin(n_ranges + 1)
    tw.insert_table(tb)
    if far:
        tw.insert((1 << 47) + 3, 4099, 0)
    n = (1 << 20) + 77
    q = make_queries(tb, n, n_ranges).numpy().view(np.uint64)
    q[:6] = [[0, 1], [U64_MAX, U64_MAX], [(1 << 47) + 3, 4099], [(1 << 47) + 4, 4099],
             [(1 << 47) + 2, 1], [int(tb.base[0]) - 1, 2]]
    assert_same(tw, q, f"{n_ranges} ranges")
    from synth.workloads import make_dma_queries
    q = make_dma_queries(tb, n, n_ranges).numpy().view(np.uint64)
    qd = torch.from_numpy(q.view(np.int64).copy()).cuda()
    v = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    o = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    tw.g.agile_validate_dma(tw.h, qd, n, v, o)
    ev, eo = tw.ot.dma_verdict_many(q[:, 0], q[:, 1])
    assert np.array_equal(v.cpu().numpy(), ev) and np.array_equal(o.cpu().numpy(), eo)
    tw.close()


def _edge_queries(base, size, seed):
    """Queries around both ends of sampled ranges, whole ranges, and lengths and addresses at the limits."""
    rng = np.random.default_rng(seed)
    k = rng.integers(0, base.size, 4000)
    k[:2] = 0, base.size - 1
    b, s = base[k], size[k]
    one = np.ones_like(b)
    sets = [(b, s), (b, s + one), (b, s - one), (b + s - one, one), (b + s, one), (b - one, one),
            (b - one, one + one), (b + s - one, one + one), (b, one * np.uint64((1 << 32) + 1)),
            (b, one * np.uint64(U64_MAX)), (b + one, s - one),
            (b + rng.integers(0, 1 << 62, b.size).astype(np.uint64) % s, rng.integers(0, 1 << 62, b.size).astype(np.uint64) % s),
            (rng.integers(0, 1 << 63, b.size).astype(np.uint64), one)]
    q = np.concatenate([np.stack(x, 1) for x in sets])
    return np.concatenate([q, np.array([[0, 1], [U64_MAX, U64_MAX], [U64_MAX, 1]], dtype=np.uint64)])


def _byte_table(form):
    """Tables above 15,100 ranges that the byte index describes, or just does not."""
    if form in ("mixed", "most", "churned"):
        return make_table({"mixed": 20000, "most": 1 << 16, "churned": 20000}[form], 2500, 3)
    rng = np.random.default_rng(5)
    n = 20001
    size, gap = {
        "256 in a bin": (np.full(n, 4096), np.full(n, 4096)),
        "no alignment": (rng.integers(1, 65, n), rng.integers(0, 16, n)),
        "largest": (rng.integers(1, 1 << 30, n), rng.integers(0, 1 << 24, n)),
        "too large": (np.where(np.arange(n) == 77, 1 << 30, 4096), np.zeros(n, np.int64)),
        "empty bins": (np.full(n, 4096), np.where(np.arange(n) % 8000 == 7, 40 << 20, 4096 * 40)),
        "too many empty bins": (np.full(n, 4096), np.where(np.arange(n) % 2000 == 7, 40 << 20, 4096 * 40)),
        "far apart": (np.full(n, 4096), np.where(np.arange(n) == 7, 1 << 32, 0)),
    }[form]
    align = {"no alignment": 1, "largest": 1 << 22}.get(form, 4096)
    step = (size + gap + align - 1) // align * align
    base = (1 << 41) + np.concatenate([[0], np.cumsum(step)[:-1]])
    kind = rng.choice([0, 0, 0, 1, 2], n)
    from synth import Table
    return Table(torch.from_numpy(base), torch.from_numpy(size.astype(np.int64)),
                 torch.from_numpy(kind.astype(np.uint8)))


@pytest.mark.parametrize("form", ["mixed", "most", "churned", "256 in a bin", "no alignment", "largest",
                                  "too large", "empty bins", "too many empty bins", "far apart"])
def test_bulk_queries_on_large_tables(form):
    """From 2^20 queries on, a large table is searched through two bytes per range, if those describe it and
    2^10 queries per range have been checked since it changed (the first calls here go the general way):
    bins with many ranges and with none, sizes of one step and of thirty powers of two, bases on any
    alignment, ids out of order, ranges too large or too far apart; pointer and DMA queries, a ragged
    count, and fewer queries on the same table."""
    need_gpu()
    from synth.workloads import make_dma_queries
    tb = _byte_table(form)
    base, size = (x.numpy().astype(np.uint64) for x in (tb.base, tb.size))
    tw = Twin(base.size)
    ids = tw.insert_table(tb)
    if form == "churned":
        for k in (100, 200):
            tw.remove(int(ids[k]))
        for k in (100, 200):
            tw.insert(int(base[k]), int(size[k]), int(tb.kind[k]))
    n = (1 << 20) + 77
    edge = _edge_queries(base, size, 9)
    q = make_queries(tb, n, 4).numpy().view(np.uint64)
    q[:edge.shape[0]] = edge
    q[-1] = edge[1]
    qd = torch.from_numpy(q.view(np.int64).copy()).cuda()
    v = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    o = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    for _ in range((base.size << 10) // n):
        tw.g.agile_validate_ptrs(tw.h, qd, n, v, o)
    assert_same(tw, q, form)
    assert_same(tw, edge, form)
    q = make_dma_queries(tb, n, 4).numpy().view(np.uint64)
    q[:edge.shape[0]] = edge
    qd = torch.from_numpy(q.view(np.int64).copy()).cuda()
    v = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    o = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    tw.g.agile_validate_dma(tw.h, qd, n, v, o)
    ev, eo = tw.ot.dma_verdict_many(q[:, 0], q[:, 1])
    assert np.array_equal(v.cpu().numpy(), ev) and np.array_equal(o.cpu().numpy(), eo)
    tw.close()
