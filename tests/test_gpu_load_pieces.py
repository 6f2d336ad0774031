"""The load-time checks over traces longer than one piece of rows (2048, one
wave each): counts that go negative in, at the edge of and after a piece, an
instant that spans the edge with the model's rows on both sides, and an
instant longer than a piece. The row in the message equals the lowest last
row of an instant with a negative count, from a cumulative sum on the host. A
trace that is one instant is refused for its range, in the time of a load."""
import re
import time

import edge_traces as E
import numpy as np
import oracle as O
import pytest
from test_gpu_parity import _cfg, _columns_from_host

pytestmark = pytest.mark.gpu
ARR, ADM, PRE, DEC, FIN = 0, 0x81, 1, 2, 3
M, WIN, NW = 5, 1000, 20


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_29160_amd import device, tre
    return tre, device, torch


def _lowest_negative(tr):
    ts, mdl, ty = tr["ts"], tr["model"], tr["type"]
    worst = None
    for m in range(M):
        r = np.flatnonzero(mdl == m)
        if not len(r):
            continue
        a = np.cumsum((ty[r] == ADM).astype(int) - (ty[r] == FIN))
        w = np.cumsum((ty[r] == ARR).astype(int) - (ty[r] == ADM))
        last = np.append(ts[r][1:] != ts[r][:-1], True)
        bad = r[last & ((a < 0) | (w < 0))]
        if len(bad):
            worst = int(bad[0]) if worst is None else min(worst, int(bad[0]))
    return worst


def _filler(n, t_max):
    """n rows over [0, t_max): whole requests of models 2 and 3, in order."""
    rows = [(0, 2 + (r // 4) % 2, 10_000 + r // 4, (ARR, ADM, DEC, FIN)[r % 4], 1) for r in range(n)]
    return [(r * t_max // n,) + row[1:] for r, row in enumerate(rows)]


def _tail(lead, kind):
    t = 9000
    out = {"finish": [(t, 0, 1, ARR, 5), (t + 1, 0, 1, FIN, 0), (t + 2, 0, 1, ADM, 5)],
           "admit": [(t, 1, 2, ADM, 5), (t + 1, 1, 2, FIN, 0)],
           "same": [(t, 1, 2, ADM, 5), (t, 1, 2, ARR, 5), (t + 1, 1, 2, FIN, 0)],
           # one instant across the edge, model 0 on both sides of it, model 1 before it only
           "span": [(t, 1, 3, ARR, 1)] + [(t, 0, 10 + k, ADM, 1) for k in range(40)] +
                   [(t, 0, 10 + k, ARR, 1) for k in range(40)],
           "span_short": [(t, 1, 3, ADM, 1)] + [(t, 0, 10 + k, ADM, 1) for k in range(40)] +
                         [(t, 0, 10 + k, ARR, 1) for k in range(39)],
           # an instant longer than a piece
           "long": [(t, 0, 10 + k, ADM, 1) for k in range(5000)] + [(t, 0, 10 + k, ARR, 1) for k in range(5000)],
           "long_short": [(t, 0, 10 + k, ADM, 1) for k in range(5000)] +
                         [(t, 0, 10 + k, ARR, 1) for k in range(4999)]}[kind]
    return out + [(t + 10 + k, 4, 90_000, DEC, 1) for k in range(200)]


@pytest.mark.parametrize("kind", ["finish", "admit", "same", "span", "span_short", "long", "long_short"])
@pytest.mark.parametrize("lead", [1968, 2007, 2044, 2048, 8190, 16384])
def test_pieces(lib, lead, kind):
    tre, device, torch = lib
    traces = [E._pack(_filler(100, 5000)), E._pack(_filler(lead, 8000) + _tail(lead, kind))]
    cols, off = _columns_from_host(torch, traces)
    row = _lowest_negative(traces[1])
    assert (row is None) == (kind in ("same", "span", "long"))
    assert O.get().trace_status(traces[1], WIN, WIN * NW, M) == (0 if row is None else -5)

    def load(req):
        tre.tre_load_events(cols["ts"], cols["model"], req, cols["type"], cols["tokens"], off,
                            _cfg(M, WIN, NW, fast_w=2, slow_w=4)).close()
    for req in (None, cols["req"]):
        if row is None:
            load(req)
            continue
        with pytest.raises(tre.TreError) as e:
            load(req)
        assert e.value.code == tre.TRE_ESTATE
        got = re.match(r".*row (\d+): an active", str(e.value))
        assert got and int(got[1]) == int(off[1]) + row, (str(e.value), int(off[1]) + row)


def test_one_instant(lib):
    """2^23 rows of one timestamp, FINISH rows first: too many for their window, and
    every piece's counts are negative to the last row. Refused without reading each
    piece's instant to its end."""
    tre, device, torch = lib
    n = 1 << 23
    ts = np.arange(n) * 20_000 // n
    ty = np.array([ARR, ADM, DEC, FIN], np.uint8)[np.arange(n) % 4]
    bad = {"ts": np.full(n, 5), "model": np.zeros(n), "req": np.zeros(n), "tokens": np.ones(n),
           "type": np.where(np.arange(n) < n // 3, FIN, np.where(np.arange(n) < 2 * n // 3, ADM, ARR))}
    good = dict(bad, ts=ts, type=ty, model=np.arange(n) // 4 % M)
    best = {}
    for name, tr in (("good", good), ("bad", bad)):
        cols, off = _columns_from_host(torch, [{k: np.asarray(v).astype(d) for k, v, d in
                                               ((k, tr[k], d) for k, d in (("ts", np.int64), ("model", np.uint8), ("req", np.uint32),
                                                                           ("type", np.uint8), ("tokens", np.uint16)))}])
        for _ in range(3):
            t0 = time.perf_counter()
            try:  # windows of 1 ms: 419 rows each
                tre.tre_load_events(cols["ts"], cols["model"], None, cols["type"], cols["tokens"], off,
                                    _cfg(M, 1, 20_000, fast_w=2, slow_w=4)).close()
                assert name == "good"
            except tre.TreError as e:
                assert name == "bad" and e.code == tre.TRE_ERANGE and "row 0:" in str(e), (name, str(e))
            best[name] = min(best.get(name, 1e9), time.perf_counter() - t0)
    assert best["bad"] < 10 * best["good"] + 0.02, best
