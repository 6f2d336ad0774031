"""Calibration of few long traces, taken by request-id records at once: at the
row count where the rule changes, with shorter and empty traces beside the
long one, ids past req_cap, and req_cap one more than the longest trace's rows
(then streamed). Traces that the stream hands over take the same kernels. Every
output equals the oracle's bit for bit."""
import numpy as np
import pytest
import tracegen as tg

import test_gpu_calib as C

pytestmark = pytest.mark.gpu
ROWS = 1 << 17


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_29160_amd import device, tre
    return tre, device, torch


def _traces(n_rows, M):
    w = tg.Workload(name="records", n_traces=2, model_classes=[["7B", "13B", "34B", "70B"][m % 4] for m in range(M)],
                    interactive=[m % 2 == 0 for m in range(M)], r_init=[2] * M, budget=2 * M, window_ms=500,
                    duration_ms=3_600_000, process="poisson", rate=[2.5] * M, seed=91)
    h = w.generate(0, 2)
    long, short = h.trace(0), h.trace(1)
    assert len(long["ts"]) >= n_rows
    cut = {k: v[:n_rows] for k, v in long.items()}  # a prefix keeps the counts and lifecycles valid
    return w, [cut, {k: v[:9000] for k, v in short.items()}, {k: v[:0] for k, v in short.items()}]


@pytest.mark.parametrize("n_rows,cap,tiers", [(ROWS, None, (0, 3)), (ROWS - 1, None, (0, 0)), (ROWS + 8193, -50, (0, 3)),
                                              (ROWS, ROWS, (0, 3)), (ROWS, ROWS + 1, (0, 0))])
def test_records(lib, n_rows, cap, tiers):
    M = 5
    w, traces = _traces(n_rows, M)
    most = C._req_cap(traces)
    assert most < n_rows
    req_cap = most if cap is None else most + cap if cap < 0 else cap
    C._check(lib, f"records {n_rows} rows, req_cap {req_cap}", w.trace_cfg(), traces, w.profile_columns(3),
             w.slo_columns(3), req_cap, tiers=tiers)


@pytest.mark.parametrize("n_listed", [1, 2, 700, 2050])
def test_listed_traces(lib, n_listed):
    """Traces that overflow both stream tiers, one to more than there are workgroups
    (2048): their records are reset and judged by all of them together."""
    over, fits = C._long_instant(4), C._turnover(400, 50)
    traces = [fits] + [over] * n_listed + [fits]
    n = len(traces)
    C._check(lib, f"{n_listed} listed", C._small_cfg(2), traces, C._small_prof(2, n), C._small_slo(2, n), C._req_cap([over, fits]),
             tiers=(n_listed, n_listed))


def test_one_trace_by_records(lib):
    w, traces = _traces(ROWS, 5)
    C._check(lib, "one trace", w.trace_cfg(), traces[:1], w.profile_columns(1), w.slo_columns(1), C._req_cap(traces[:1]),
             tiers=(0, 1))
