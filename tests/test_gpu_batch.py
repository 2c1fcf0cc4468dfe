"""Batched multi-client requests (one persistent launch) against the oracle.

Four clients, each with its own table (synthetic ranges plus a real device arena holding a
copy source, a protected canary, a hole, a gather table, an index buffer and one output slot
per request). Requests mix pointer validation (own-table, cross-client and hostile pointers)
with guarded copies or gathers, several of them hostile. Checked: every pointer's verdict and
owner, every request's lowest failing argument, the arenas byte for byte, every request's fault
record; then each request run alone gives the same result as in the mix.
"""
import random

import numpy as np
import pytest
import torch

from gpu_util import need_gpu, guard_mod
from oracle import guarded as G
from oracle.batched import batch_verdicts
from oracle.memory import Memory
from oracle.table import RangeTable as OracleTable
from synth import make_table, make_queries

pytestmark = pytest.mark.gpu

ARENA = 1 << 20
SRC, PROT, HOLE, GT, IDX, SLOTS = 0, 128 << 10, 132 << 10, 136 << 10, 392 << 10, 520 << 10
SLOT = 16 << 10
NSLOT = (ARENA - SLOTS) // SLOT


class Client:
    def __init__(self, g, c, n_ranges=200):
        self.tb = make_table(n_ranges, n_ranges // 5, 100 + c, first_hi=2**44)
        self.rt = g.RangeTable(n_ranges + 312)
        self.ot = OracleTable()
        self.rt.insert_many(self.tb.base, self.tb.size, self.tb.kind)
        for b, s, k in zip(self.tb.base.tolist(), self.tb.size.tolist(), self.tb.kind.tolist()):
            self.ot.insert(b, s, k)
        gen = torch.Generator().manual_seed(1000 + c)
        host = torch.randint(0, 256, (ARENA,), dtype=torch.uint8, generator=gen)
        rows = (IDX - GT) // 4
        idx = torch.randint(0, rows, ((SLOTS - IDX) // 8,), generator=gen)
        bad = torch.randperm(idx.numel(), generator=gen)[:idx.numel() // 20]
        idx[bad] = torch.tensor([rows, rows + 7, -1, -(1 << 40), (PROT - GT) // 4 + 3, 1 << 62],
                                dtype=torch.int64)[torch.arange(bad.numel()) % 6]
        host[IDX:SLOTS] = idx.view(torch.uint8)
        self.dev = host.cuda()
        self.base = self.dev.data_ptr()
        self.mem = Memory()
        self.mem.add(self.base, host.numpy())
        regions = [(SRC, PROT, 0), (PROT, HOLE, 1), (GT, IDX, 0), (IDX, SLOTS, 0)]
        regions += [(SLOTS + k * SLOT, SLOTS + (k + 1) * SLOT, 0) for k in range(NSLOT)]
        for lo, hi, kind in regions:
            a = self.rt.insert(self.base + lo, hi - lo, kind)
            b = self.ot.insert(self.base + lo, hi - lo, kind)
            assert a == b

    def a(self, off):
        return self.base + off


def build(seed, ncl=4, nreq=40, n_ranges=200):
    g = guard_mod()
    cls = [Client(g, c, n_ranges) for c in range(ncl)]
    rng = random.Random(seed)
    reqs = np.zeros(nreq, dtype=g.REQUEST_DTYPE)
    ptrs = []
    slot_of = {c: 0 for c in range(ncl)}
    for r in range(nreq):
        c = r % ncl
        cl = cls[c]
        other = cls[(c + 1) % ncl]
        m = rng.choice([0, 1, 3, 50, 700, 3000])
        q = make_queries(cl.tb, max(m, 1), seed * 1000 + r).numpy()[:m].tolist()
        for k in range(len(q)):
            u = rng.random()
            if u < 0.1:
                q[k] = [cl.a(SLOTS + rng.randrange(0, SLOT)), rng.choice([1, 8, 64])]
            elif u < 0.15:
                q[k] = [other.a(SRC + 64), 16]                # valid only for another client
            elif u < 0.18:
                q[k] = [cl.a(PROT + 8), 8]
        reqs[r]["client"] = c
        reqs[r]["ptr_off"] = len(ptrs)
        reqs[r]["nptr"] = len(q)
        ptrs += q
        slot = SLOTS + slot_of[c] * SLOT
        slot_of[c] += 1
        kind = rng.random()
        if kind < 0.6:
            reqs[r]["copy_dst"] = cl.a(slot) if rng.random() < 0.85 else cl.a(HOLE)
            src = rng.choice([cl.a(SRC + rng.randrange(0, 4096)), cl.a(SRC + 120 * 1024),
                              cl.a(PROT), other.a(SRC), cl.a(SRC + 3)])
            reqs[r]["copy_src"] = src
            reqs[r]["copy_bytes"] = rng.choice([1, 15, 4096, 12345, SLOT, SLOT + 100])
        elif kind < 0.9:
            rbytes = rng.choice([4, 8])
            n = rng.choice([1, 100, 2000, SLOT // rbytes, SLOT // rbytes + 3])
            reqs[r]["gather_out"] = cl.a(slot)
            reqs[r]["gather_table"] = cl.a(GT)
            reqs[r]["gather_idx"] = cl.a(IDX + 8 * rng.randrange(0, 1000))
            reqs[r]["gather_n"] = n
            reqs[r]["gather_row_bytes"] = rbytes
    P = torch.tensor(np.array(ptrs, dtype=np.uint64).reshape(-1, 2).view(np.int64)).cuda() \
        if ptrs else torch.zeros((1, 2), dtype=torch.int64, device="cuda")
    return g, cls, reqs, P, len(ptrs)


def run_batch(g, cs, reqs, P, nptrs):
    pv = torch.full((max(nptrs, 1),), 255, dtype=torch.uint8, device="cuda")
    po = torch.full((max(nptrs, 1),), -7, dtype=torch.int32, device="cuda")
    res = torch.zeros(len(reqs) * g.RESULT_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    g.agile_batch_run(cs, reqs, P, nptrs, pv, po, res)
    torch.cuda.synchronize()
    return pv.cpu().numpy()[:nptrs], po.cpu().numpy()[:nptrs], g.batch_results(res, len(reqs))


def oracle_request(cl, q, r):
    log = G.FaultLog()
    if q["copy_bytes"]:
        G.copy_vec(cl.ot, cl.mem, log, r, int(q["copy_dst"]), int(q["copy_src"]),
                   int(q["copy_bytes"]))
    if q["gather_n"]:
        G.gather_vec(cl.ot, cl.mem, log, r, int(q["gather_out"]), int(q["gather_table"]),
                     int(q["gather_row_bytes"]), int(q["gather_idx"]), int(q["gather_n"]), 4)
    return log


def check_fault(res, log, r, seq):
    assert res["count"] == log.count, (r, res, log.count)
    if log.count == 0:
        assert res["first_seq"] == (1 << 64) - 1
        return
    f = log.first
    got = dict(elem=int(res["first_elem"]), operand=int(res["first_operand"]),
               addr=int(res["first_addr"]), width=int(res["first_width"]),
               verdict=int(res["first_verdict"]), owner=int(res["first_owner"]),
               op=int(res["first_op"]))
    want = {k: f[k] for k in got}
    assert got == want and int(res["first_seq"]) == seq, (r, got, want)


@pytest.mark.parametrize("seed,n_ranges", [(1, 200), (2, 200), (3, 200), (4, 9000),
                                            (5, 20000), (6, 8192 - 4 - NSLOT),
                                            (7, 8193 - 4 - NSLOT)])
def test_batch_against_oracle_and_alone_identity(seed, n_ranges):
    """Client tables of 200 ranges have their bucket splitters staged in LDS; tables of 9,000
    and 20,000 ranges (more than 4,096 buckets) are searched in global memory; tables of exactly
    8,192 ranges (4,096 buckets, the most that are staged) and 8,193 (the fewest searched in
    global memory) sit on either side of the boundary."""
    need_gpu()
    g, cls, reqs, P, nptrs = build(seed, n_ranges=n_ranges)
    counts = [len(cl.rt) for cl in cls]
    assert all(c == n_ranges + 4 + NSLOT for c in counts), counts
    if n_ranges > 8192:
        assert min(counts) > 8192, counts   # more than 4,096 buckets: the unstaged search
    cs = g.agile_clients_create([cl.rt for cl in cls])
    pv, po, res = run_batch(g, cs, reqs, P, nptrs)
    # pointer verdicts and per-request lowest failing argument
    ev, eo, rv, ra, ro = batch_verdicts([cl.ot for cl in cls], reqs["client"],
                                        np.append(reqs["ptr_off"], nptrs).astype(np.int64),
                                        P.cpu().numpy()[:nptrs].view(np.uint64))
    assert np.array_equal(pv, ev) and np.array_equal(po, eo)
    assert np.array_equal(res["verdict"], rv) and np.array_equal(res["arg"], ra)
    assert np.array_equal(res["owner"], ro) and (res["done"] == 1).all()
    # data movement and fault records, request by request in the oracle
    for r, q in enumerate(reqs):
        log = oracle_request(cls[int(q["client"])], q, r)
        check_fault(res[r], log, r, r)
    for c, cl in enumerate(cls):
        got = cl.dev.cpu().numpy()
        assert np.array_equal(got, cl.mem.buffer(cl.base)), f"client {c} arena differs"
        assert (got[PROT:HOLE] == cl.mem.buffer(cl.base)[PROT:HOLE]).all()
    # each request alone equals its result in the mix (outputs rewritten with the same bytes)
    for r in range(len(reqs)):
        one = reqs[r:r + 1].copy()
        p1, o1, r1 = run_batch(g, cs, one, P, nptrs)
        a, b = int(reqs[r]["ptr_off"]), int(reqs[r]["ptr_off"] + reqs[r]["nptr"])
        assert np.array_equal(p1[a:b], pv[a:b]) and np.array_equal(o1[a:b], po[a:b])
        for k in ("verdict", "arg", "owner", "count", "first_elem", "first_operand",
                  "first_addr", "first_verdict", "first_owner"):
            assert r1[0][k] == res[r][k], (r, k)
    for c, cl in enumerate(cls):
        assert np.array_equal(cl.dev.cpu().numpy(), cl.mem.buffer(cl.base))
    g.agile_clients_destroy(cs)


@pytest.mark.parametrize("src_off,dst_off", [(0, 0), (5, 0), (0, 3), (4, 9), (15, 1)])
def test_batch_copies_at_the_edges_of_tiles(src_off, dst_off):
    """Copies around a workgroup's pass (32 KiB) and a tile (128 KiB), with the source and the
    destination at any place in a 16-byte vector, whole and with either end denied, against the
    oracle byte for byte and in their fault records."""
    need_gpu()
    g = guard_mod()
    sizes = [1, 15, 16, 17, 32767, 32768, 32784, 131071, 131072, 131073, 300001]
    cap = max(sizes) + 64
    n = len(sizes) * 3
    gen = torch.Generator().manual_seed(src_off * 16 + dst_off)
    host = torch.randint(0, 256, (cap * (n + 1) + 4096,), dtype=torch.uint8, generator=gen)
    dev = host.cuda()
    mem, ot, rt = Memory(), OracleTable(), g.RangeTable(n * 2 + 8)
    mem.add(dev.data_ptr(), host.numpy())
    base = dev.data_ptr() + (-dev.data_ptr()) % 16
    reqs = np.zeros(n, dtype=g.REQUEST_DTYPE)
    src_end = base + src_off + 200_000      # the source's range ends inside the largest copies
    ranges = [(base, src_end - base)]
    for r in range(n):
        size, cut = sizes[r // 3], (r % 3) * 9      # destination: whole, 9 or 18 bytes short
        lo = base + cap * (r + 1)
        lo += -lo % 16 + dst_off
        if size > cut:
            ranges.append((lo, size - cut))
        reqs[r]["copy_src"], reqs[r]["copy_dst"], reqs[r]["copy_bytes"] = base + src_off, lo, size
    for b, s in ranges:
        rt.insert(b, s, 0)
        ot.insert(b, s, 0)
    cs = g.agile_clients_create([rt])
    _, _, res = run_batch(g, cs, reqs, torch.zeros((1, 2), dtype=torch.int64, device="cuda"), 0)
    assert (res["done"] == 1).all()
    for r, q in enumerate(reqs):
        log = G.FaultLog()
        G.copy_vec(ot, mem, log, r, int(q["copy_dst"]), int(q["copy_src"]), int(q["copy_bytes"]))
        check_fault(res[r], log, r, r)
    assert np.array_equal(dev.cpu().numpy(), mem.buffer(dev.data_ptr()))
    g.agile_clients_destroy(cs)


@pytest.mark.parametrize("n_ranges,align", [(4096, 4096), (4100, 1), (8192, 4096), (8196, 4096),
                                            (16400, 1)])
def test_batch_pointers_with_keys_of_either_width(n_ranges, align):
    """Tables whose bucket keys fit 32 bits (page-aligned bases) and tables whose keys do not
    (byte-granular bases over a wide span), with the most buckets that are staged whole and a few
    more, against the oracle at and around every range's ends."""
    need_gpu()
    g = guard_mod()
    rng = random.Random(n_ranges + align)
    ot, rt = OracleTable(), g.RangeTable(n_ranges)
    pos, q = (1 << 41) + (0 if align > 1 else 3), []
    for k in range(n_ranges):
        pos += rng.randrange(0, 4) * align + (rng.randrange(1 << 24) if align == 1 else 0)
        size = rng.choice([1, 7, align, 3 * align])
        kind = rng.choice([0, 0, 1, 2])
        rt.insert(pos, size, kind)
        ot.insert(pos, size, kind)
        q += [[pos - 1, 2], [pos, size], [pos + size - 1, 1], [pos + size, 1]]
        pos += size + (-size) % align
    q += [[0, 1], [(1 << 64) - 1, 1], [1 << 41, 0]]
    qn = np.array(q, dtype=np.uint64)
    cs = g.agile_clients_create([rt])
    reqs = np.zeros(1, dtype=g.REQUEST_DTYPE)
    reqs[0]["nptr"] = len(q)
    pv, po, res = run_batch(g, cs, reqs, torch.from_numpy(qn.view(np.int64)).cuda(), len(q))
    ev, eo = ot.verdict_many(qn[:, 0], qn[:, 1])
    assert np.array_equal(pv, ev) and np.array_equal(po, eo)
    assert res[0]["arg"] == int(np.flatnonzero(ev)[0]) and res[0]["done"] == 1
    g.agile_clients_destroy(cs)


@pytest.mark.parametrize("n", [133119, 133120, 266239, 266240, 300001])
def test_batch_gathers_around_the_growth_of_their_tiles(n):
    """Gather tiles double while the largest gather has more than 64: both sides of each step, beside
    gathers that end inside a tile, every hundredth index hostile, against torch and the denials' count."""
    need_gpu()
    g = guard_mod()
    rows, gen = 5000, torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(rows + 64, generator=gen, device="cuda")
    sizes = [n, 1, 2047, 2049, 8193, 65537]
    idx = torch.randint(0, rows, (sum(sizes),), generator=gen, device="cuda")
    idx[torch.rand(sum(sizes), generator=gen, device="cuda") < 0.01] = rows + 5
    out = torch.full((sum(sizes),), 7.0, device="cuda")
    rt = g.RangeTable(16)
    for x in (buf[:rows], idx, out):
        rt.insert_tensor(x)
    reqs, at = np.zeros(len(sizes), dtype=g.REQUEST_DTYPE), 0
    for r, k in enumerate(sizes):
        reqs[r]["gather_out"], reqs[r]["gather_table"] = out.data_ptr() + 4 * at, buf.data_ptr()
        reqs[r]["gather_idx"], reqs[r]["gather_n"] = idx.data_ptr() + 8 * at, k
        reqs[r]["gather_row_bytes"] = 4
        at += k
    cs = g.agile_clients_create([rt])
    for few in (False, True):
        out.fill_(7.0)
        q = reqs[:1] if few else reqs
        _, _, res = run_batch(g, cs, q, torch.zeros((1, 2), dtype=torch.int64, device="cuda"), 0)
        assert (res["done"] == 1).all()
        m = n if few else sum(sizes)
        ok = idx[:m] < rows
        want = torch.where(ok, buf[idx[:m].clamp(max=rows - 1)], torch.zeros((), device="cuda"))
        assert torch.equal(out[:m], want) and bool((out[m:] == 7.0).all())
        denied = [int((~p).sum()) for p in ok.split(sizes[:1] if few else sizes)]
        assert [int(x) for x in res["count"]] == denied
    g.agile_clients_destroy(cs)


@pytest.mark.parametrize("rb", [12, 16, 20, 60, 64, 68, 1020, 1024, 1028])
def test_batch_gathers_of_wide_rows(rb):
    """Rows of 16 bytes and more move in vectors, the last one overlapping: every width of a lane group and
    several passes of a wave, tiles' remainders, hostile indices, an index buffer and an output that end
    before the rows do, against the oracle byte for byte and in their fault records."""
    need_gpu()
    g = guard_mod()
    D, rows, sizes = rb // 4, 37, [1, 63, 513, 2049]
    gen = torch.Generator().manual_seed(rb)
    span = [k * rb + 64 for k in sizes]
    host = torch.randint(0, 256, (rows * rb + 64 + 2 * sum(span),), dtype=torch.uint8, generator=gen)
    dev = host.cuda()
    hidx = torch.randint(0, rows, (sum(sizes) * 2,), generator=gen)
    hidx[torch.rand(hidx.shape, generator=gen) < 0.05] = rows + 3
    hidx[torch.rand(hidx.shape, generator=gen) < 0.02] = -(1 << 62)
    didx = hidx.cuda()
    mem, ot, rt = Memory(), OracleTable(), g.RangeTable(64)
    mem.add(dev.data_ptr(), host.numpy())
    mem.add(didx.data_ptr(), hidx.numpy().view(np.uint8))
    base = dev.data_ptr()
    ranges, at, ia = [(base, rows * rb)], base + rows * rb + 64, didx.data_ptr()
    reqs = np.zeros(2 * len(sizes), dtype=g.REQUEST_DTYPE)
    for r in range(2 * len(sizes)):
        n, cut = sizes[r // 2], r % 2           # every other request: buffers that end early
        ranges.append((at, max(4, n * rb - cut * (2 * rb - 4))))
        ranges.append((ia, 8 * max(1, n - cut)))
        reqs[r]["gather_out"], reqs[r]["gather_table"], reqs[r]["gather_idx"] = at, base, ia
        reqs[r]["gather_n"], reqs[r]["gather_row_bytes"] = n, rb
        at += n * rb + 64 - (n * rb + 64) % 4
        ia += 8 * n
    for b, s in ranges:
        rt.insert(b, s, 0)
        ot.insert(b, s, 0)
    cs = g.agile_clients_create([rt])
    _, _, res = run_batch(g, cs, reqs, torch.zeros((1, 2), dtype=torch.int64, device="cuda"), 0)
    assert (res["done"] == 1).all()
    for r, q in enumerate(reqs):
        log = G.FaultLog()
        G.gather_vec(ot, mem, log, r, int(q["gather_out"]), base, rb, int(q["gather_idx"]), int(q["gather_n"]), 4)
        check_fault(res[r], log, r, r)
    assert np.array_equal(dev.cpu().numpy(), mem.buffer(dev.data_ptr()))
    g.agile_clients_destroy(cs)
