"""The token check with arrays at the least alignment that it takes (tokens 8 bytes, clients and slots 4,
kinds and verdicts 1): pairs of tokens are loaded and stored together from wherever they lie. Against
the oracle, with the bytes around the outputs left alone, for both record layouts, with and without the
slot records in LDS."""
import numpy as np
import pytest
import torch

from gpu_util import guard_mod, need_gpu
from oracle import tokens as T

pytestmark = pytest.mark.gpu

KEY = 0x0F1E2D3C4B5A6978


@pytest.mark.parametrize("big_owner", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 1023, 1024, 2047, 100_001, (1 << 21) + 3])
def test_token_check_at_odd_addresses(n, big_owner):
    need_gpu()
    g = guard_mod()
    slots = 3000
    ts, ot = g.TokenTable(slots, KEY), T.TokenTable(slots, KEY)
    rng = np.random.default_rng(n)
    owner = rng.integers(0, 50, slots // 2) + ((1 << 30) if big_owner else 0)
    kind = rng.integers(0, 4, slots // 2)
    tok = np.array([ts.mint(int(o), int(k)) for o, k in zip(owner, kind)], np.uint64)
    for t, o, k in zip(tok, owner, kind):
        assert int(t) == ot.mint(int(o), int(k))
    for i in rng.choice(slots // 2, 200, replace=False):
        ts.release(int(tok[i]), int(owner[i]))
        ot.release(int(tok[i]), int(owner[i]))
    pick = rng.integers(0, tok.size, n)
    tokens, clients, kinds = tok[pick], owner[pick].astype(np.uint32), kind[pick].astype(np.uint8)
    u = rng.random(n)
    tokens = np.where(u < 0.1, tokens ^ np.uint64(1 << 9), tokens)
    clients[(u > 0.1) & (u < 0.2)] += 1
    kinds[(u > 0.2) & (u < 0.3)] = 7
    kinds[(u > 0.3) & (u < 0.4)] = T.ANY_KIND

    def place(a, off):
        b = torch.zeros(a.nbytes + off + 64, dtype=torch.uint8, device="cuda")
        b[off:off + a.nbytes] = torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).copy()).cuda()
        return b, b.data_ptr() + off

    for to, co, ko, vo, so in ((8, 4, 1, 1, 4), (0, 0, 3, 0, 12), (8, 12, 0, 5, 0), (0, 4, 7, 3, 4)):
        (tb, tp), (cb, cp), (kb, kp) = place(tokens, to), place(clients, co), place(kinds, ko)
        for with_kinds in (True, False):
            vb = torch.full((vo + n + 64,), 0xAA, dtype=torch.uint8, device="cuda")
            sb = torch.full((so // 4 + n + 16,), -77, dtype=torch.int32, device="cuda")
            g.agile_tokens_check(ts.handle, tp, cp, kp if with_kinds else None, n, vb.data_ptr() + vo,
                                 sb.data_ptr() + so)
            ev, es = T.check_many(ot, tokens.tolist(), clients.tolist(), kinds.tolist() if with_kinds else None)
            v, s = vb.cpu().numpy(), sb.cpu().numpy()
            assert np.array_equal(v[vo:vo + n], ev) and np.array_equal(s[so // 4:so // 4 + n], es)
            assert (v[:vo] == 0xAA).all() and (v[vo + n:] == 0xAA).all()
            assert (s[:so // 4] == -77).all() and (s[so // 4 + n:] == -77).all()
    ts.close()
