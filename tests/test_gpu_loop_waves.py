"""The closed loop with several waves per scenario: the scenario counts where
the number of waves changes (and where one wave per scenario takes over), model
counts that do not divide among the waves, heaps too large for the LDS at their
full sizes (one wave again), slots per replica that are no multiple of 4, more
starts in a window than a request ring or the list of starts holds, and a
backlog. Against the oracle, every output bit for bit."""
import numpy as np
import pytest
import tracegen as tg

import test_gpu_loop as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_29160_amd import device, tre
    return tre, device, torch


def _run(lib, M, n_sc, duration_s, rate=0.8, window_ms=500, spr=8, r_cap=16, act=False, extra=3):
    w = tg.Workload(name=f"waves-{M}-{n_sc}", n_traces=1, model_classes=[["7B", "13B", "34B", "70B"][m % 4] for m in range(M)],
                    interactive=[m % 2 == 0 for m in range(M)], r_init=[2] * M, budget=2 * M + extra,
                    window_ms=window_ms, duration_ms=1000 * duration_s, process="mmpp2", rate=[rate] * M,
                    proc_params={"mmpp_mult": 6.0, "mmpp_dwell_s": 60.0}, seed=70 + M)
    rng = np.random.default_rng(M + n_sc)
    cfg = dict(w.trace_cfg())
    a = None
    if act:
        fp, veto = L._act_model(rng, 1, M, L._n_ticks(cfg))
        cfg["budget"] = int(2 * fp.sum()) + extra
        a = (1310, 1870, fp, veto)
    L._check(lib, w.name, cfg, [w.requests(0)], w.profile_columns(1), w.slo_columns(1), w.service_columns(1),
             L._scenarios(rng, n_sc, 1, ks=(1, 2, 4, 0)), spr=spr, r_cap=r_cap, act=a)


@pytest.mark.parametrize("n_sc", [256, 257, 513, 1025, 2048, 2049])
def test_scenario_counts(lib, n_sc):
    _run(lib, 9, n_sc, 30)
    if n_sc > 1024:
        _run(lib, 3, n_sc, 20, act=True)


@pytest.mark.parametrize("M", [2, 3, 7, 8, 9, 33, 63])
def test_model_counts(lib, M):
    _run(lib, M, 3, 200)
    _run(lib, M, 3, 100, act=True)


def test_large_heaps(lib):
    """1024 slots per model: 256 KiB for 64 models, 128 KiB for 32."""
    _run(lib, 64, 2, 60, spr=16, r_cap=64, extra=8)
    _run(lib, 32, 2, 60, spr=16, r_cap=64, extra=8)


@pytest.mark.parametrize("spr", [1, 3, 6])
def test_slots_and_backlog(lib, spr):
    """Rates far above what the slots serve: requests wait over many windows."""
    _run(lib, 5, 4, 120, rate=6.0, spr=spr, act=spr == 3)


def test_starts_beyond_the_rings(lib):
    """More arrivals and starts of one model in a 5 s window than a ring holds."""
    _run(lib, 2, 3, 200, rate=12.0, window_ms=5000, spr=64)
    _run(lib, 20, 600, 40, rate=12.0, window_ms=5000, spr=32, r_cap=8)


@pytest.mark.parametrize("minutes,M,n_sc,act", [(20, 8, 4, False), (30, 8, 4, True), (30, 3, 4, False), (30, 1, 2049, True)])
def test_long_windows(lib, minutes, M, n_sc, act):
    """One model's finishes of one window, each up to minutes before its end,
    sum to more than 32 bits hold: with several waves, with one wave a scenario,
    and (2049 scenarios) in the kernel for many scenarios."""
    W = minutes * 60_000
    w = tg.standard(1).scaled(name=f"long-{minutes}min-{M}", model_classes=["7B"] * M, interactive=[m % 2 == 0 for m in range(M)],
                              r_init=[4] * M, budget=4 * M, rate=[9.0] * M, prompt_mu=[5.0] * M, out_mu=[3.5] * M, process="poisson",
                              duration_ms=2 * W, window_ms=W, fast_period_ms=W, slow_period_ms=W)
    tables = [w.requests(0)]
    a = np.asarray(tables[0]["arrival_ms"])
    # a request is done within a minute of its arrival at this load
    te = np.maximum(W - a % W - 60_000, 0) * (a < W)
    assert max(int(te[tables[0]["model"] == m].sum()) for m in range(M)) > 1 << 32
    rng = np.random.default_rng(minutes + M)
    cfg = dict(w.trace_cfg())
    model = None
    if act:
        fp, veto = L._act_model(rng, 1, M, L._n_ticks(cfg))
        cfg["budget"] = int(4 * fp.sum()) + 3
        model = (1310, 1870, fp, veto)
    L._check(lib, w.name, cfg, tables, w.profile_columns(1), w.slo_columns(1), w.service_columns(1),
             L._scenarios(rng, n_sc, 1, ks=(1, 2, 4, 0)), act=model)
