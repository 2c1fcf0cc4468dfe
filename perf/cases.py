"""Workloads of the range guard, one dict each, with what is needed to time them.

``listed()`` names twelve workloads from one mediated request to the sizes of the full benchmark,
``draw(rng)`` gives further ones of the same ranges, ``prepare(case, seed)`` makes what a caller
holds before the call (tables, inputs, output buffers), ``run(state)`` is one pass through the
public entry points, ``work(case)`` the bytes and operations that the pass cannot do without, and
``exact(case, seed)`` the floating-point outputs in 64 bits by plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_06697_amd import guard as g
from paper_2606_06697_amd.embedding import guarded_embedding
from synth.workloads import (make_dma_queries, make_queries, make_table, uniform_f32,
                             uniform_indices, zipf_indices)

DEV = "cuda"
PAD = 16          # protected rows right behind a row table: what hostile indices aim at
SCALE = 3.0       # the triad's scalar
KEY = 0x5DEECE66D  # secret key of the token tables


def listed():
    return [
        # one mediated request: its pointer arguments against the calling client's table
        dict(name="ptrs_request", op="validate", n=200, ranges=4096, dma=False),
        # the DMA registration check of a client with the serving mix's largest table
        dict(name="dma_mid", op="validate", n=1_000_003, ranges=8192, dma=True),
        # bulk validation against the largest table
        dict(name="ptrs_large", op="validate", n=(1 << 26) + 77, ranges=65536, dma=False),
        # the smallest guarded copy of a request (launch latency)
        dict(name="copy_small", op="copy", nbytes=4096, src_off=0, dst_off=0),
        # an odd-sized copy out of the middle of a packed byte buffer
        dict(name="copy_ragged", op="copy", nbytes=(64 << 20) + 13, src_off=5, dst_off=0),
        # streaming triad over buffers far larger than the last-level cache
        dict(name="triad_large", op="triad", n=(1 << 27) + 3, off=0),
        # random single-element gather over a 1 GiB table, 0.1% hostile indices
        dict(name="gather_random", op="gather", rows=1 << 28, D=1, n=(1 << 25) + 1, f64=False,
             zipf=False, bad=1e-3),
        # a small training batch through the guarded embedding, forward and backward
        dict(name="embed_small", op="embed", rows=4096, D=64, n=5000, f64=False, bad=1e-2),
        # an ordinary training batch
        dict(name="embed_mid", op="embed", rows=4096, D=32, n=50_000, f64=False, bad=1e-2),
        # the largest embedding: a 1 GiB table, a million Zipf-distributed indices
        dict(name="embed_large", op="embed", rows=1 << 20, D=256, n=1 << 20, f64=False, bad=1e-4),
        # handle tokens of many clients, presented in bulk
        dict(name="tokens_large", op="tokens", slots=1 << 20, n=(1 << 24) + 5, kinds=True),
        # one batched launch over many clients: pointers, guarded copies and guarded gathers
        dict(name="batch_large", op="batch", clients=16, ranges=4096, nreq=512, max_ptrs=4096,
             max_copy=16 << 20, max_gather=1 << 16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    op = rng.choice(["validate", "validate", "copy", "triad", "gather", "scatter", "embed", "embed",
                     "tokens", "batch"])
    if op == "validate":
        return dict(op=op, n=_log_int(rng, 16, 1 << 26), ranges=_log_int(rng, 64, 65536),
                    dma=rng.random() < 0.3)
    if op == "copy":
        s, d = rng.choice([(0, 0), (0, 0), (4, 0), (8, 8), (rng.randrange(16), rng.randrange(16))])
        return dict(op=op, nbytes=_log_int(rng, 4096, 256 << 20), src_off=s, dst_off=d)
    if op == "triad":
        return dict(op=op, n=_log_int(rng, 1 << 12, 1 << 27), off=rng.choice([0, 0, 1, 3]))
    f64 = rng.random() < 0.25
    if op == "gather":
        D = _log_int(rng, 1, 512)
        rows = _log_int(rng, 256, max(256, (1 << 28) // D // (2 if f64 else 1)))
        n = _log_int(rng, 64, max(64, (1 << 27) // max(D, 4) // (2 if f64 else 1)))
        return dict(op=op, rows=rows, D=D, n=n, f64=f64, zipf=rng.random() < 0.3,
                    bad=rng.choice([0.0, 1e-3, 1e-2]))
    if op == "scatter":
        D = _log_int(rng, 1, 256)
        rows = _log_int(rng, 256, 1 << 20)
        n = _log_int(rng, 64, 1 << 19)
        add = rng.random() < 0.7
        return dict(op=op, rows=rows if add else max(rows, n), D=D, n=n, f64=f64, add=add,
                    bad=rng.choice([0.0, 1e-3, 1e-2]))
    if op == "embed":
        return dict(op=op, rows=_log_int(rng, 256, 1 << 20), D=_log_int(rng, 2, 256),
                    n=_log_int(rng, 64, 1 << 19), f64=f64, bad=rng.choice([0.0, 1e-4, 1e-2]))
    if op == "tokens":
        return dict(op=op, slots=_log_int(rng, 256, 1 << 20), n=_log_int(rng, 64, 1 << 24),
                    kinds=rng.random() < 0.7)
    return dict(op=op, clients=rng.randint(1, 16), ranges=_log_int(rng, 1024, 8192),
                nreq=_log_int(rng, 1, 512), max_ptrs=_log_int(rng, 64, 4096),
                max_copy=_log_int(rng, 1 << 16, 16 << 20), max_gather=_log_int(rng, 1 << 12, 1 << 16))


# ---- inputs -------------------------------------------------------------------------------
def _dtype(case):
    return torch.float64 if case["f64"] else torch.float32


def _values(n, seed, stream, dtype):
    """Values uniform in [-1, 1) of either type."""
    if dtype == torch.float32:
        return uniform_f32(n, seed, DEV, stream)
    gen = torch.Generator(device=DEV).manual_seed(seed * 1_000_003 + stream)
    return torch.rand(n, generator=gen, device=DEV, dtype=dtype) * 2.0 - 1.0


def _offset(nbytes, off, fill=None):
    """A byte view at `off` bytes behind a 256-byte boundary."""
    buf = torch.zeros(nbytes + off, dtype=torch.uint8, device=DEV)
    if fill is not None:
        buf[off:off + nbytes] = fill
    return buf[off:off + nbytes]


def _row_inputs(case, seed):
    """A row table with protected rows behind it, the indices into it and one row per index."""
    rows, D, n, dt = case["rows"], case["D"], case["n"], _dtype(case)
    buf = torch.empty((rows + PAD) * D, dtype=dt, device=DEV)
    buf[:rows * D] = _values(rows * D, seed, 31, dt)
    buf[rows * D:] = 0
    bad = ((rows, rows + PAD),)
    if case["op"] == "scatter" and not case["add"]:  # distinct rows: the result has one value
        gen = torch.Generator(device=DEV).manual_seed(seed + 17)
        idx = torch.randperm(rows, generator=gen, device=DEV)[:n].contiguous()
        idx[torch.rand(n, generator=gen, device=DEV) < case["bad"]] = rows + 1
    elif case["op"] in ("embed", "scatter") or case["zipf"]:
        idx = zipf_indices(n, rows, 1.1, seed, DEV, case["bad"], bad)
    else:
        idx = uniform_indices(n, rows, seed, DEV, case["bad"], bad)
    src = None if case["op"] == "gather" else _values(n * D, seed, 32, dt).view(n, D)
    return buf, idx, src


def _row_table(buf, rows, D, idx):
    rt = g.RangeTable(64)
    table, pad = buf[:rows * D].view(rows, D), buf[rows * D:]
    rt.insert_tensor(table)
    rt.insert_tensor(pad, g.KIND_PROTECTED)
    rt.insert_tensor(idx)
    return rt, table


def _batch_state(case, seed):
    """Clients with their tables, gather tables and copy sources, and one launch's requests; every
    request writes into its own registered output."""
    gen = np.random.default_rng(case["nreq"])  # the sizes; what the buffers hold is the seed's
    ncl, nreq = case["clients"], case["nreq"]

    def log_ints(lo, hi, n):
        v = np.exp(gen.uniform(math.log(lo), math.log(hi + 1), n)).astype(np.int64)
        return np.clip(v, lo, hi)

    client = gen.integers(0, ncl, nreq)
    nptr = log_ints(1, case["max_ptrs"], nreq)
    gather = gen.random(nreq) < 0.2
    copy_bytes = np.where(gather, 0, log_ints(4096, case["max_copy"], nreq))
    gather_n = np.where(gather, log_ints(1024, case["max_gather"], nreq), 0)
    need = (np.where(gather, gather_n * 4, copy_bytes) + 255) // 256 * 256
    out = torch.zeros(int(need.sum()), dtype=torch.uint8, device=DEV)
    out_at = np.concatenate([[0], np.cumsum(need)])[:-1]
    tabs, srcs, gtabs, idxs, ptrs = [], [], [], [], []
    for c in range(ncl):
        tb = make_table(case["ranges"], case["ranges"] // 8, seed * 64 + c, first_hi=2**44)
        rt = g.RangeTable(case["ranges"] + nreq + 16)
        rt.insert_many(tb.base, tb.size, tb.kind)
        tg = torch.Generator(device=DEV).manual_seed(seed * 64 + c)
        src = torch.randint(0, 256, (case["max_copy"],), generator=tg, dtype=torch.uint8, device=DEV)
        buf = torch.rand((1 << 20) + PAD, generator=tg, device=DEV)
        gt, pad = buf[:1 << 20], buf[1 << 20:]
        rt.insert_tensor(pad, g.KIND_PROTECTED)
        ix = uniform_indices(case["max_gather"], 1 << 20, seed * 64 + c, DEV, 1e-3,
                             ((1 << 20, (1 << 20) + PAD),))
        for t in (src, gt, ix):
            rt.insert_tensor(t)
        tabs.append(rt), srcs.append(src), gtabs.append(gt), idxs.append(ix)
        if (client == c).any():
            ptrs.append(make_queries(tb, int(nptr[client == c].sum()), seed * 64 + c, DEV))
    reqs = np.zeros(nreq, g.REQUEST_DTYPE)
    reqs["client"], reqs["nptr"] = client, nptr
    at = np.concatenate([[0], np.cumsum([nptr[client == c].sum() for c in range(ncl)])])[:-1]
    for r in range(nreq):
        c = int(client[r])
        reqs[r]["ptr_off"] = at[c]
        at[c] += nptr[r]
        dst = out.data_ptr() + int(out_at[r])
        tabs[c].insert(dst, int(need[r]), g.KIND_USER, backed=True)
        if gather[r]:
            reqs[r]["gather_out"], reqs[r]["gather_table"] = dst, gtabs[c].data_ptr()
            reqs[r]["gather_idx"], reqs[r]["gather_n"] = idxs[c].data_ptr(), gather_n[r]
            reqs[r]["gather_row_bytes"] = 4
        else:
            reqs[r]["copy_dst"], reqs[r]["copy_src"] = dst, srcs[c].data_ptr()
            reqs[r]["copy_bytes"] = copy_bytes[r]
    ptrs = torch.cat(ptrs).contiguous()
    m = ptrs.shape[0]
    return dict(op="batch", set=_Clients(tabs), reqs=reqs, ptrs=ptrs, nptrs=m, out=out,
                verdict=torch.zeros(m, dtype=torch.uint8, device=DEV),
                owner=torch.zeros(m, dtype=torch.int32, device=DEV),
                result=torch.zeros(nreq, 18, dtype=torch.int32, device=DEV),
                keep=(srcs, gtabs, idxs))


class _Clients:
    """A client set, destroyed before the tables that it is made of."""

    def __init__(self, tables):
        self.tables, self.handle = tables, g.agile_clients_create(tables)

    def __del__(self):
        g.agile_clients_destroy(self.handle)


def _token_inputs(case, seed):
    """A slot table half in use by 64 clients and what is presented to it: mostly live tokens, the
    rest released, of another client or made up."""
    n, live, ncl = case["n"], max(8, case["slots"] // 2), 64
    ts = g.TokenTable(case["slots"], KEY + seed)
    gen = np.random.default_rng(seed)
    owner = gen.integers(0, ncl, live)
    kind = gen.integers(0, 4, live)
    tok = np.array([ts.mint(int(o), int(k)) for o, k in zip(owner, kind)], np.uint64)
    for k in gen.choice(live, live // 8, replace=False):
        ts.release(int(tok[k]), int(owner[k]))
    tg = torch.Generator(device=DEV).manual_seed(seed)
    pick = torch.randint(0, live, (n,), generator=tg, device=DEV)
    tokens = torch.from_numpy(tok.view(np.int64)).to(DEV)[pick]
    clients = torch.from_numpy(owner.astype(np.int32)).to(DEV)[pick]
    kinds = torch.from_numpy(kind.astype(np.uint8)).to(DEV)[pick]
    u = torch.rand(n, generator=tg, device=DEV)
    tokens = torch.where(u < 0.05, tokens ^ 0x5A5A, tokens)
    clients = torch.where((u >= 0.05) & (u < 0.13), (clients + 1) % ncl, clients)
    return dict(op="tokens", ts=ts, tokens=tokens, clients=clients, kinds=kinds if case["kinds"] else None)


# ---- what a caller holds, one pass, its work and its exact result -------------------------
def prepare(case, seed):
    op = case["op"]
    if op == "validate":
        tb = make_table(case["ranges"], case["ranges"] // 8, seed)
        rt = g.RangeTable(case["ranges"])
        rt.insert_many(tb.base, tb.size, tb.kind)
        n = case["n"]
        q = (make_dma_queries if case["dma"] else make_queries)(tb, n, seed, DEV)
        return dict(op="dma" if case["dma"] else "ptrs", rt=rt, q=q, n=n,
                    verdict=torch.empty(n, dtype=torch.uint8, device=DEV),
                    owner=torch.empty(n, dtype=torch.int32, device=DEV))
    if op == "copy":
        n = case["nbytes"]
        gen = torch.Generator(device=DEV).manual_seed(seed)
        data = torch.randint(0, 256, (n,), generator=gen, dtype=torch.uint8, device=DEV)
        src, dst = _offset(n, case["src_off"], data), _offset(n, case["dst_off"])
        rt = g.RangeTable(64)
        rt.insert_tensor(src), rt.insert_tensor(dst)
        return dict(op=op, rt=rt, src=src, dst=dst, n=n)
    if op == "triad":
        n, o = case["n"], case["off"]
        b, c = (uniform_f32(n + o, seed, DEV, k)[o:] for k in (33, 34))
        a = torch.zeros(n + o, device=DEV)[o:]
        rt = g.RangeTable(64)
        for t in (a, b, c):
            rt.insert_tensor(t)
        return dict(op=op, rt=rt, a=a, b=b, c=c, n=n)
    if op == "tokens":
        return _token_inputs(case, seed)
    if op == "batch":
        return _batch_state(case, seed)
    rows, D, n = case["rows"], case["D"], case["n"]
    buf, idx, src = _row_inputs(case, seed)
    rt, table = _row_table(buf, rows, D, idx)
    st = dict(op=op, rt=rt, buf=buf, table=table, idx=idx, src=src, n=n,
              rb=D * buf.element_size(), dt=g.DTYPE_F64 if case["f64"] else g.DTYPE_F32)
    if op == "embed":
        st["table"] = table.requires_grad_()
    elif op == "gather":
        st["out"] = torch.zeros(n, D, dtype=buf.dtype, device=DEV)
        rt.insert_tensor(st["out"])
    else:
        st["add"] = g.SCATTER_ADD if case["add"] else g.SCATTER
        rt.insert_tensor(src)
    return st


def run(st):
    op = st["op"]
    if op == "ptrs":
        g.agile_validate_ptrs(st["rt"].handle, st["q"], st["n"], st["verdict"], st["owner"])
        return [st["verdict"], st["owner"]]
    if op == "dma":
        g.agile_validate_dma(st["rt"].handle, st["q"], st["n"], st["verdict"], st["owner"])
        return [st["verdict"], st["owner"]]
    if op == "copy":
        g.agile_guarded_copy(st["rt"].handle, st["dst"], st["src"], st["n"])
        return [st["dst"]]
    if op == "triad":
        g.agile_guarded_triad(st["rt"].handle, st["a"], st["b"], st["c"], SCALE, st["n"])
        return [st["a"]]
    if op == "gather":
        g.agile_guarded_gather(st["rt"].handle, st["out"], st["table"], st["rb"], st["idx"],
                               st["n"], st["dt"])
        return [st["out"]]
    if op == "scatter":
        g.agile_guarded_scatter(st["rt"].handle, st["table"], st["rb"], st["idx"], st["src"],
                                st["n"], st["dt"], st["add"])
        return [st["table"]]
    if op == "embed":
        y = guarded_embedding(st["table"], st["idx"], st["rt"])
        (dw,) = torch.autograd.grad(y, st["table"], st["src"])
        return [y, dw]
    if op == "tokens":
        return list(st["ts"].check(st["tokens"], st["clients"], st["kinds"]))
    g.agile_batch_run(st["set"].handle, st["reqs"], st["ptrs"], st["nptrs"], st["verdict"], st["owner"],
                      st["result"])
    res = st["result"]  # without a fault's address, which is where this process has the buffer
    return [st["out"], st["verdict"], st["owner"], res[:, :10], res[:, 12:]]


def _distinct(case):
    """Expected number of distinct rows that the indices name."""
    rows, n = case["rows"], case["n"]
    if case["op"] == "scatter" and not case["add"]:
        return n
    if case["op"] in ("embed", "scatter") or case["zipf"]:
        p = torch.arange(1, rows + 1, dtype=torch.float64).pow(-1.1)
        p /= p.sum()
        return float((1.0 - (1.0 - p).pow(n)).sum())
    return rows * -math.expm1(-n / rows)


def work(case):
    op = case["op"]
    if op == "validate":
        return dict(bytes=21 * case["n"], flops=0)
    if op == "copy":
        return dict(bytes=2 * case["nbytes"], flops=0)
    if op == "triad":
        return dict(bytes=12 * case["n"], flops=2 * case["n"])
    if op == "tokens":
        return dict(bytes=(18 if case["kinds"] else 17) * case["n"] + 4 * case["slots"], flops=0)
    if op == "batch":  # log-uniform sizes: their mean is (hi - lo) / log(hi / lo)
        def mean(lo, hi):
            return (hi - lo) / math.log(hi / lo)
        per = 21 * mean(1, case["max_ptrs"]) + 0.8 * 2 * mean(4096, case["max_copy"]) \
            + 0.2 * 16 * mean(1024, case["max_gather"])
        return dict(bytes=case["nreq"] * per, flops=0)
    rows, D, n = case["rows"], case["D"], case["n"]
    rb = D * (8 if case["f64"] else 4)
    hit = _distinct(case) * rb
    if op == "gather":
        return dict(bytes=8 * n + hit + n * rb, flops=0)
    if op == "scatter":
        return dict(bytes=8 * n + n * rb + (2 if case["add"] else 1) * hit,
                    flops=n * D if case["add"] else 0)
    # forward: indices, the rows they name, the output; backward: dY in, dW out
    return dict(bytes=8 * n + hit + 2 * n * rb + rows * rb, flops=n * D)


def exact(case, seed):
    op = case["op"]
    if op == "triad":
        n, o = case["n"], case["off"]
        b, c = (uniform_f32(n + o, seed, DEV, k)[o:].double() for k in (33, 34))
        return [b.add_(c, alpha=SCALE)]
    if op not in ("gather", "scatter", "embed"):
        return None  # whole numbers and bytes only
    rows, D, n = case["rows"], case["D"], case["n"]
    buf, idx, src = _row_inputs(case, seed)
    table = buf[:rows * D].view(rows, D).double()
    ok = (idx >= 0) & (idx < rows)
    if op != "scatter":
        y = table[idx.clamp(0, rows - 1)]
        y[~ok] = 0
        if op == "gather":
            return [y]
        return [y, torch.zeros_like(table).index_add_(0, idx[ok], src[ok].double())]
    if case["add"]:
        return [table.index_add_(0, idx[ok], src[ok].double())]
    table[idx[ok]] = src[ok].double()
    return [table]
