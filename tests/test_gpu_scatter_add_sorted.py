"""Guarded scatter-add on the sorted path, which calls of more than 2^18 rows take: every combination that
its key, sort, reduce and exact-row kernels tell apart, against the oracle. The arena and its
integer values are those of test_gpu_scatter_add.py, whose cases of 32,768 to 70,001 rows are added
chunk by chunk: every sum is exact in any order, and the arena must equal the oracle's memory byte for
byte. The widths cover one, two and four elements a lane, and rows of a part of a wave and of more."""
import numpy as np
import pytest

import test_gpu_redirect
import test_gpu_scatter_add as base
import test_gpu_trap
from gpu_util import Arena, Twin, log_matches, need_gpu
from oracle import guarded as G

pytestmark = pytest.mark.gpu

N = (1 << 18) + 257     # the last tile, chunk and histogram are partial
ROWS = base.DST_ROWS


def setup(w, D, seed, monkeypatch, rows=ROWS, more_ranges=0):
    monkeypatch.setattr(base, "NMAX", N)
    need_gpu()
    off, size = base.layout(w, D, rows)
    ar = Arena(size, seed)
    tw = Twin(16 + more_ranges)
    for k, kind in {"dst": 0, "prot": 1, "other": 0, "idx": 0, "src": 0}.items():
        lo, hi = off[k]
        tw.insert(ar.addr(lo), hi - lo, kind)
    for k in range(more_ranges):    # elsewhere: the finishing kernel reads the uploaded table
        tw.insert((1 << 20) + 8192 * k, 4096, 1)
    rng = np.random.default_rng(seed)
    for k in ("dst", "src", "other"):
        lo, hi = off[k]
        ar.write(lo, rng.integers(-50, 51, (hi - lo) // w).astype(np.float32 if w == 4 else np.float64))
    return ar, tw, off


def both(ar, tw, ol, w, rb, dst, idx, src, n, what, accumulate=1, policy=G.SUPPRESS_LOG):
    tw.g.agile_guarded_scatter(tw.h, dst, rb, idx, src, n, 0 if w == 4 else 1, accumulate, policy)
    G.scatter_vec(tw.ot, ar.mem, ol, tw.next_seq(), dst, rb, idx, src, n, w, True, policy)
    ar.check(what)
    log_matches(tw, ol, what)


def numbers(rng, n, rows, extra, neg=0):
    """Hot rows, uniform rows and hostile values."""
    hot = rng.integers(0, rows, 5)
    bad = np.array([rows, rows + 1, -1 - neg, 3 * rows, -(1 << 62), 1 << 62, -(1 << 63), (1 << 63) - 1,
                    (1 << 40) + 3, *extra], dtype=np.int64)
    u, v = rng.random(n), rng.integers(-neg, rows, n)
    v[u < 0.5] = hot[np.minimum(rng.exponential(1.0, n).astype(np.int64), 4)][u < 0.5]
    v[u > 0.9] = bad[rng.integers(0, bad.size, n)][u > 0.9]
    return v.astype(np.int64)


@pytest.mark.parametrize("w,D", [(4, 1), (4, 3), (4, 20), (4, 64), (4, 100), (8, 2), (8, 33)])
def test_sorted_path_where_pointers_end_or_are_interior_or_unbound(w, D, monkeypatch):
    ar, tw, off = setup(w, D, 900 + D + w, monkeypatch)
    rb, ol, rng = w * D, G.FaultLog(), np.random.default_rng(901 + D + w)
    dst = ar.addr(off["dst"][0])
    extra = [(ar.addr(off[k][0]) - dst) // rb + 1 for k in ("prot", "hole", "other")]
    (ilo, ihi), (slo, shi) = off["idx"], off["src"]
    trials = [("plain", dst, ar.addr(ilo), ar.addr(slo), 0),
              ("index and source end before n", dst, ar.addr(ihi - 8 * (N - 700)),
               ar.addr(shi - rb * (N - 1234) - w), 0),
              ("interior destination", dst + 100 * rb + w, ar.addr(ilo), ar.addr(slo), 100),
              ("unbound destination", ar.addr(off["hole"][0]), ar.addr(ilo), ar.addr(slo), 0)]
    for what, d, ip, sp, neg in trials:
        idx = numbers(rng, N, ROWS - 101 if neg else ROWS, extra, neg)
        ar.write(ip - ar.base, idx[:(ihi - (ip - ar.base)) // 8])
        both(ar, tw, ol, w, rb, d, ip, sp, N, f"w={w} D={D} {what}")
    tw.close()


@pytest.mark.parametrize("w,D,rows", [(4, 4, 256), (4, 1, 65536), (8, 1, 256), (4, 20, 256)])
def test_sorted_path_whose_last_pass_sees_one_digit(w, D, rows, monkeypatch):
    """2^8 or 2^16 rows and no hostile one: the last pass is skipped, and the reduce reads the buffer of the
    one before. Then into zeros."""
    ar, tw, off = setup(w, D, 950 + D + w, monkeypatch, rows=rows)
    rb, ol, rng = w * D, G.FaultLog(), np.random.default_rng(rows + w)
    a = [ar.addr(off[k][0]) for k in ("dst", "idx", "src")]
    for accumulate in (1, 2):
        if accumulate == 2:
            ar.write(off["dst"][0], np.zeros(rows * rb // 4, np.int32))
        idx = rng.integers(0, rows, N)
        idx[rng.random(N) < 0.3] = rows - 1
        ar.write(off["idx"][0], idx.astype(np.int64))
        both(ar, tw, ol, w, rb, a[0], a[1], a[2], N, f"{rows} rows, accumulate {accumulate}", accumulate)
    tw.close()


@pytest.mark.parametrize("w,D", [(4, 64), (4, 3), (8, 2), (4, 130)])
def test_sorted_path_of_the_unguarded_twin(w, D, monkeypatch):
    ar, tw, off = setup(w, D, 970 + D, monkeypatch)
    rb = w * D
    rng = np.random.default_rng(971 + D)
    idx = numbers(rng, N, ROWS, [])
    idx[(idx < 0) | (idx >= ROWS)] = 7
    ar.write(off["idx"][0], idx)
    a = [ar.addr(off[k][0]) for k in ("dst", "idx", "src")]
    tw.g.agile_unguarded_scatter(a[0], rb, a[1], a[2], N, 0 if w == 4 else 1, 1)
    G.scatter_vec(tw.ot, ar.mem, G.FaultLog(), 0, a[0], rb, a[1], a[2], N, w, True)
    ar.check("unguarded sorted scatter-add")
    assert tw.rt.fault_log()[1]["count"] == 0
    # and with negative rows of an interior destination, whose keys lie below 2^31
    ar.write(off["idx"][0], idx - 100)
    interior = a[0] + 100 * rb
    tw.g.agile_unguarded_scatter(interior, rb, a[1], a[2], N, 0 if w == 4 else 1, 1)
    G.scatter_vec(tw.ot, ar.mem, G.FaultLog(), 0, interior, rb, a[1], a[2], N, w, True)
    ar.check("unguarded sorted scatter-add, interior destination")
    tw.close()


@pytest.mark.parametrize("more_ranges", [0, 70])
@pytest.mark.parametrize("w,D", [(4, 20), (8, 2)])
def test_sorted_path_policies_and_tables_beyond_the_launch_arguments(w, D, more_ranges, monkeypatch):
    """SUPPRESS_ONLY leaves the log empty and takes its number; the logged call after it records with the
    next one. With more than 64 ranges the denials are recorded by a kernel after the launch. The call
    without allocation is the same."""
    ar, tw, off = setup(w, D, 990 + D + more_ranges, monkeypatch, more_ranges=more_ranges)
    rb, ol, rng = w * D, G.FaultLog(), np.random.default_rng(991 + D)
    a = [ar.addr(off[k][0]) for k in ("dst", "idx", "src")]
    ar.write(off["idx"][0], numbers(rng, N, ROWS, [(ar.addr(off["prot"][0]) - a[0]) // rb + 1]))
    for policy in (G.SUPPRESS_ONLY, G.SUPPRESS_LOG):
        both(ar, tw, ol, w, rb, *a, N, f"policy {policy}, {more_ranges} more ranges", policy=policy)
    tw.g.agile_guarded_scatter_add_noalloc(tw.h, *a[:1], rb, *a[1:], N, 0 if w == 4 else 1)
    G.scatter_vec(tw.ot, ar.mem, ol, tw.next_seq(), a[0], rb, a[1], a[2], N, w, True)
    ar.check("without allocation")
    log_matches(tw, ol, "without allocation")
    # no row denied, then every row
    for what, idx in (("none denied", rng.integers(0, ROWS, N)), ("all denied", np.full(N, ROWS + 1))):
        ar.write(off["idx"][0], idx.astype(np.int64))
        both(ar, tw, ol, w, rb, *a, N, what)
    tw.close()


def test_sorted_path_under_the_trap_policy(monkeypatch):
    monkeypatch.setattr(test_gpu_trap, "NIDX", N)
    test_gpu_trap.test_trap_on_the_sorted_scatter_add_path()


@pytest.mark.parametrize("policy", [G.SINK, G.REPORT, G.REMAP])
def test_sorted_path_under_the_redirecting_policies(policy, monkeypatch):
    # the source ends 512 bytes behind a multiple of the quarantine's size, as with 40,000 rows
    n = (1 << 18) + 64
    monkeypatch.setattr(test_gpu_redirect, "NMAX", n)
    test_gpu_redirect.test_scatter_add_redirected(policy, n)
