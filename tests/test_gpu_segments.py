"""GPU parity of the segmented path of the streaming kernels (few traces: the
windows of a trace cut into segments, then one chain over the raw ratios) and
of the prepared ticks of the control replay, at the sizes where they can go
wrong: columns at the edges of the chain's two forms (16 and 17 models, 8 and
9 for the two shares of a stage), windows one more or less than a chunk or a
segment, fewer windows than a chunk, every window a tick, more moves per tick
than models, and the number of scenarios at which the replay changes kernels.
Every per-cell output, decision and replica sum equals the oracle's bit for
bit. A sweep captured in a graph takes no scratch of the library's pool; its
replays equal the eager call."""
import numpy as np
import pytest

import parity as PT
import test_gpu_parity as P
import test_gpu_stage as S
import tracegen as tg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_29160_amd import device, tre
    return tre, device, torch


def _workload(M, n_windows, n_traces, window_ms, seed, fast_w, slow_w):
    classes = [["7B", "13B", "34B", "70B"][m % 4] for m in range(M)]
    return tg.standard(1).scaled(
        name=f"seg-{M}m-{n_windows}w-{n_traces}t", n_traces=n_traces, model_classes=classes,
        interactive=[m % 2 == 0 for m in range(M)], r_init=[2 + m % 3 for m in range(M)], budget=3 * M + 2,
        window_ms=window_ms, duration_ms=n_windows * window_ms, rate=[0.3 + 0.4 * (m % 5) for m in range(M)],
        fast_period_ms=fast_w * window_ms, slow_period_ms=slow_w * window_ms, seed=seed)


@pytest.mark.parametrize("M,n_windows,n_traces,window_ms,fast_w,slow_w", [
    (1, 33, 1, 1000, 1, 2), (3, 31, 2, 500, 2, 3), (8, 64, 1, 500, 10, 20), (8, 65, 3, 250, 1, 1),
    (16, 257, 2, 200, 5, 7), (17, 129, 2, 200, 5, 15), (32, 63, 3, 250, 4, 8), (33, 40, 2, 250, 3, 4),
    (64, 19, 2, 500, 1, 3), (5, 48, 160, 500, 4, 8), (5, 48, 161, 500, 4, 8)])
def test_edges(lib, M, n_windows, n_traces, window_ms, fast_w, slow_w):
    w = _workload(M, n_windows, n_traces, window_ms, 1000 + M, fast_w, slow_w)
    evs = w.generate(0, n_traces)
    traces = [evs.trace(i) for i in range(n_traces)]
    prof = w.profile_columns(n_traces)
    rng = np.random.default_rng(M)
    n = n_traces + (1 if n_traces > 1 else 0)  # one trace carries two scenarios
    sc = {"trace": (np.arange(n) % n_traces).astype(np.uint32),
          "max_moves": rng.choice(np.array([1, 3, 70], np.uint32), n).astype(np.uint32),
          "theta_scale": rng.uniform(0.5, 2.0, n), "tau_crit_override": rng.uniform(0.2, 0.8, n)}
    P._check_set(lib, w.name, w.trace_cfg(), traces, prof, sc)
    S._check(lib, w.name, w.trace_cfg(), traces, prof)


def test_stage_columns(lib):
    """8 and 9 models: 16 and 18 share columns."""
    for M in (8, 9):
        w = _workload(M, 100, 3, 500, 7 + M, 10, 20)
        evs = w.generate(0, 3)
        S._check(lib, w.name, w.trace_cfg(), [evs.trace(i) for i in range(3)], w.profile_columns(3))


@pytest.mark.parametrize("n_sc", [2048, 2049])
def test_scenario_counts(lib, n_sc):
    """One trace, the replay in prepared ticks and in folds."""
    w = _workload(6, 60, 1, 500, 3, 2, 4)
    evs = w.generate(0, 1)
    sc = P._random_scenarios(1, n_sc, 11)
    P._check_set(lib, f"{n_sc} scenarios", w.trace_cfg(), [evs.trace(0)], w.profile_columns(1), sc)


def test_captured_sweep(lib):
    tre, device, torch = lib
    w = _workload(8, 200, 4, 250, 21, 4, 8)
    dt = device.upload(w)
    ev = device.load(dt)
    prof = device.profiles(w)
    sc = device.scenarios(P._random_scenarios(4, 6, 5))
    cap = ev.n_ticks * 8
    ws = torch.empty(tre.tre_workspace_size(ev, 6), dtype=torch.uint8, device="cuda")

    def outputs():
        return tre.ctl_outputs(ev, 6, cap), torch.zeros((4, ev.n_windows, 8), dtype=torch.float32, device="cuda")

    ref, t32 = outputs()
    tre.tre_sweep(ev, prof, sc, ref, ws, tss32=t32)
    torch.cuda.synchronize()
    got, g32 = outputs()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):  # the kernels are loaded before the capture
        tre.tre_sweep(ev, prof, sc, got, ws, tss32=g32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        tre.tre_sweep(ev, prof, sc, got, ws, tss32=g32)
    for _ in range(3):
        for t in (got["moves"], got["n_moves"], got["r_final"], got["r_windows"], g32):
            t.zero_()
        tre.tre_sweep(ev, prof, sc, ref, ws, tss32=t32)  # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for k in ("moves", "n_moves", "r_final", "r_windows"):
            assert torch.equal(got[k], ref[k]), k
        assert torch.equal(g32.view(torch.int32), t32.view(torch.int32))
    ev.close()
