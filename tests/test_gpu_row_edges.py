"""Guarded gather and scatter of rows at the edges of their allocation, against the oracle: rows with a
few bytes inside it, the rows next to those, and rows far outside, for table pointers that do not lie
a whole number of rows from the allocation's ends, with outputs, sources and index arrays that end
inside a row. Row widths below, at and above a 16-byte vector, a group of lanes and a wave."""
import numpy as np
import pytest
import torch

from gpu_util import Arena, Twin, guard_mod, log_matches, need_gpu
from oracle import guarded as G

pytestmark = pytest.mark.gpu

ROWS = 40


def _setup(w, D, seed):
    need_gpu()
    rb = w * D
    off, o = {}, 0
    for name, size, kind in (("before", 8 * rb, 1), ("table", ROWS * rb + w, 0), ("after", 8 * rb, 1),
                             ("idx", 8 * 200, 0), ("cont", 60 * rb + 3 * w, 0), ("rest", 80 * rb, 1)):
        off[name] = (o, o + size, kind)
        o += size if name != "table" else size + (-size) % 8
    ar = Arena((o + 4095) // 4096 * 4096, seed)
    tw = Twin(16)
    for lo, hi, kind in off.values():
        tw.insert(ar.addr(lo), hi - lo, kind)
    return ar, tw, off


@pytest.mark.parametrize("w,D", [(4, 1), (4, 2), (4, 3), (4, 4), (4, 5), (4, 17), (4, 64), (4, 65), (4, 130),
                                 (4, 257), (8, 1), (8, 2), (8, 3), (8, 33), (8, 65), (8, 130)])
def test_rows_around_the_ends_of_their_allocation(w, D):
    ar, tw, off = _setup(w, D, 40 + w + D)
    rb, dtype, ol = w * D, 0 if w == 4 else 1, G.FaultLog()
    rng = np.random.default_rng(w + D)
    lo, hi, _ = off["table"]
    base0 = ar.addr(lo)
    for shift in (0, 3 * rb, 2 * rb + w * (D // 2), w, 5 * rb + (rb - w)):
        first, rows = -(shift // rb) - 3, (hi - lo) // rb + 6   # three rows past either end
        pool = np.concatenate([np.arange(first, first + rows), [-(1 << 62), (1 << 62), -(1 << 63), (1 << 63) - 1,
                                                                1 << 40, -(1 << 40)]])
        idx = rng.permutation(pool).astype(np.int64)
        n = idx.size
        for cut in ("none", "cont", "idx"):
            ilo = off["idx"][0] if cut != "idx" else off["idx"][1] - 8 * (n - 7)
            clo = off["cont"][0] if cut != "cont" else off["cont"][1] - (n - 9) * rb - w * (D // 2)
            room = (off["idx"][1] - ilo) // 8
            ar.write(ilo, idx[:room])
            args = (base0 + shift, rb, ar.addr(ilo), ar.addr(clo), n)
            what = f"w={w} D={D} shift={shift} cut={cut}"
            tw.g.agile_guarded_gather(tw.h, args[3], args[0], rb, args[2], n, dtype)
            G.gather_vec(tw.ot, ar.mem, ol, tw.next_seq(), args[3], args[0], rb, args[2], n, w)
            ar.check("gather " + what)
            log_matches(tw, ol, "gather " + what)
            # distinct rows only (an unreadable index counts as row 0): the result has one value
            m = n if cut != "idx" else room
            tw.g.agile_guarded_scatter(tw.h, args[0], rb, args[2], args[3], m, dtype, 0)
            G.scatter_vec(tw.ot, ar.mem, ol, tw.next_seq(), args[0], rb, args[2], args[3], m, w, False)
            ar.check("scatter " + what)
            log_matches(tw, ol, "scatter " + what)
    tw.close()


@pytest.mark.parametrize("add", [False, True])
@pytest.mark.parametrize("w,D,n", [(4, 1, 5000), (4, 3, 300_000), (4, 5, 100_000), (4, 17, 5000), (4, 17, 200_000),
                                   (4, 65, 40_000), (4, 255, 30_000), (8, 3, 100_000), (8, 33, 50_000),
                                   (8, 129, 20_000)])
def test_hostile_scatter_leaves_what_lies_around_its_table_alone(w, D, n, add):
    """Distinct rows and rows just outside, in calls of every number of rows in flight: the bytes before and
    behind the table are what they were, bit for bit."""
    need_gpu()
    g = guard_mod()
    dt = torch.float32 if w == 4 else torch.float64
    rows, pad = n + 100, 16
    gen = torch.Generator(device="cuda").manual_seed(w + D + n)
    buf = torch.randn((rows + 2 * pad) * D, generator=gen, device="cuda", dtype=dt)
    table = buf[pad * D:(rows + pad) * D].view(rows, D)
    src = torch.randn(n, D, generator=gen, device="cuda", dtype=dt)
    idx = torch.randperm(rows, generator=gen, device="cuda")[:n].contiguous()
    bad = torch.rand(n, generator=gen, device="cuda") < 0.05
    idx[bad] = torch.where(torch.rand(int(bad.sum()), generator=gen, device="cuda") < 0.5, rows + 3, -2)
    rt = g.RangeTable(8)
    for t in (table, src, idx):
        rt.insert_tensor(t)
    before = buf.clone()
    g.agile_guarded_scatter(rt.handle, table, D * w, idx, src, n, 0 if w == 4 else 1, int(add))
    want = before[pad * D:(rows + pad) * D].view(rows, D).clone()
    good = ~bad
    want[idx[good]] = want[idx[good]] + src[good] if add else src[good]   # one addition a row: exact
    assert torch.equal(table, want)
    bits = torch.int32 if w == 4 else torch.int64
    for part in (slice(0, pad * D), slice((rows + pad) * D, None)):
        assert torch.equal(buf[part].view(bits), before[part].view(bits))
    assert rt.fault_log()[1]["count"] == int(bad.sum()) * D
    rt.close()
