"""The fault log of calls on several streams and in graphs. Calls on one handle have to be ordered, so what
the log holds of two that overlap is not looked at; but it must not spoil the ordered calls that
follow. Calls captured in a graph log the denials of every replay."""
import pytest
import torch

from gpu_util import guard_mod, need_gpu

pytestmark = pytest.mark.gpu


class _Rows:
    def __init__(self, n, D, rows, nbad, seed):
        self.g = guard_mod()
        gen = torch.Generator(device="cuda").manual_seed(seed)
        self.n, self.rb, self.rows, self.nbad = n, 4 * D, rows, nbad
        self.table = torch.rand(rows, D, generator=gen, device="cuda")
        self.out = torch.zeros(n, D, device="cuda")
        self.good = torch.randint(0, rows, (n,), generator=gen, device="cuda")
        self.bad = self.good.clone()
        self.bad[torch.randperm(n, generator=gen, device="cuda")[:nbad]] = rows + 1

    def register(self, rt):
        for t in (self.table, self.out, self.good, self.bad):
            rt.insert_tensor(t)

    def gather(self, rt, idx, stream=None, policy=0):
        self.g.agile_guarded_gather(rt.handle, self.out, self.table, self.rb, idx, self.n, 0, policy, stream)

    def add(self, rt, idx, stream=None):
        self.g.agile_guarded_scatter(rt.handle, self.table, self.rb, idx, self.out, self.n, 0,
                                     self.g.SCATTER_ADD, 0, stream)

    def denied(self):
        return self.nbad * self.rb // 4


def test_calls_that_overlap_leave_later_ordered_calls_alone():
    need_gpu()
    g = guard_mod()
    # 1,024 and 512 workgroups, and one of a few
    a, b, c = _Rows(1 << 20, 1, 1 << 20, 700, 1), _Rows(1 << 19, 1, 1 << 18, 3, 2), _Rows(5000, 64, 4096, 11, 3)
    rt = g.RangeTable(32)
    for x in (a, b, c):
        x.register(rt)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for rep in range(12):
        for k in range(3):
            a.gather(rt, a.good, s1)
            b.gather(rt, b.good, s2)
            if rep % 3 == 0:
                c.gather(rt, c.good, s1)
        torch.cuda.synchronize()
        # the log is read, not cleared: clearing must not be what puts things right
        before = rt.fault_log()[1]["count"]
        assert before == rep * (a.denied() + b.denied() + c.denied() + 2 * c.denied())
        for x in (a, b, c):
            x.gather(rt, x.bad)
        c.add(rt, c.bad)
        c.add(rt, c.bad)
        assert rt.fault_log()[1]["count"] - before == a.denied() + b.denied() + 3 * c.denied(), rep
    # and a violation under the trap policy is seen
    with pytest.raises(g.AgileError):
        a.gather(rt, a.bad, None, g.POLICY_TRAP)
    rt.close()


def test_every_replay_of_a_graph_logs_its_denials():
    need_gpu()
    g = guard_mod()
    a, c = _Rows(1 << 19, 1, 1 << 18, 5, 4), _Rows(5000, 64, 4096, 11, 5)
    rt = g.RangeTable(32)
    for x in (a, c):
        x.register(rt)
    a.gather(rt, a.good)
    c.add(rt, c.good)
    torch.cuda.synchronize()
    c.table.zero_()
    c.out.fill_(0.5)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.gather(rt, a.bad)
        c.add(rt, c.bad)
    want_a = torch.where((a.bad < a.rows)[:, None], a.table[a.bad.clamp(max=a.rows - 1)], 0.0)
    adds = torch.bincount(c.bad[c.bad < c.rows], minlength=c.rows).float()[:, None] * 0.5
    total = 0
    for rep in range(1, 8):
        a.out.fill_(7.0)
        graph.replay()
        total += a.denied() + c.denied()
        torch.cuda.synchronize()
        assert torch.equal(a.out, want_a)
        assert torch.equal(c.table, (adds * rep).expand_as(c.table))
        assert rt.fault_log()[1]["count"] == total, rep
        if rep % 2:
            a.gather(rt, a.bad)  # the program's own calls in between
            total += a.denied()
        if rep == 4:
            assert rt.fault_log(clear=True)[1]["count"] == total
            total = 0
    rt.close()
