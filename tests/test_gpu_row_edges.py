"""Guarded gather and scatter of rows at the edges of their allocation, against the oracle: rows with a
few bytes inside it, the rows next to those, and rows far outside, for table pointers that do not lie
a whole number of rows from the allocation's ends, with outputs, sources and index arrays that end
inside a row. Row widths below, at and above a 16-byte vector, a group of lanes and a wave."""
import numpy as np
import pytest

from gpu_util import Arena, Twin, log_matches, need_gpu
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
