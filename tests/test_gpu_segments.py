"""GPU parity of the segmented path of the streaming kernels (few traces: the
windows of a trace cut into segments, then one chain over the raw ratios) and
of the prepared ticks of the control replay, at the sizes where they can go
wrong: columns at the edges of the chain's two forms (16 and 17 models, 8 and
9 for the two shares of a stage), windows one more or less than a chunk or a
segment, fewer windows than a chunk, every window a tick, more moves per tick
than models, and the number of scenarios at which the replay changes kernels.
Every per-cell output, decision and replica sum equals the oracle's bit for
bit. A sweep captured in a graph takes no scratch of the library's own; its
replays equal the eager call. The scratch is kept and given back within its
bounds and shared by no two calls of several threads and streams."""
import edge_traces as E
import numpy as np
import pytest

import parity as PT
import test_gpu_actuation as A
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


# the numbers of chunks, windows and traces at which the path changes, and (161
# and 400 traces) rows of a chunk on either side of the line
@pytest.mark.parametrize("M,n_windows,n_traces,window_ms", [
    (2, 96, 3, 500), (2, 97, 3, 500), (3, 64, 2, 500), (3, 65, 2, 500), (40, 39, 2, 200), (40, 40, 2, 200),
    (16, 48, 2, 250), (16, 49, 2, 250), (5, 130, 160, 500), (5, 130, 161, 500), (17, 41, 96, 100), (17, 41, 97, 100),
    (64, 44, 161, 500), (64, 44, 400, 1000)])
def test_rule_edges(lib, M, n_windows, n_traces, window_ms):
    test_edges(lib, M, n_windows, n_traces, window_ms, 4, 8)


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


@pytest.mark.parametrize("M,n_sc,act", [(16, 1536, True), (16, 1537, True), (17, 1024, False), (24, 1025, True), (25, 768, True),
                                        (32, 769, False), (33, 1, False), (33, 512, True), (40, 513, False), (41, 256, True),
                                        (41, 257, False), (64, 3, True), (64, 256, False)])
def test_replay_rule(lib, M, n_sc, act):
    """The models and scenarios at which the replay changes kernels, every window
    a tick."""
    w = _workload(M, 50, 1, 500, M, 1, 2)
    evs = w.generate(0, 1)
    sc = P._random_scenarios(1, n_sc, 11)
    if not act:
        P._check_set(lib, f"{M} models {n_sc} scenarios", w.trace_cfg(), [evs.trace(0)], w.profile_columns(1), sc)
        return
    rng = np.random.default_rng(M)
    g = rng.integers(1, 3, (1, M)).astype(np.int32)
    cfg = dict(w.trace_cfg(), budget=int((g[0] * np.asarray(w.r_init)).sum()) + 3)
    veto = rng.integers(0, 1 << 63, (1, 50), dtype=np.int64).astype(np.uint64) & np.uint64((1 << M) - 1)
    veto[rng.random(veto.shape) > 0.2] = 0
    A._check(lib, f"{M} models {n_sc} scenarios", cfg, [evs.trace(0)], w.profile_columns(1), sc, 1310, 1870, g, veto)


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


def _same(got, ref, what):
    """Equal bit for bit, any NaN equal to any other."""
    got, ref = np.asarray(got), np.asarray(ref)
    ok = (got == ref) | (np.isnan(got) & np.isnan(ref)) if ref.dtype.kind == "f" else got == ref
    assert ok.all(), f"{what}: {np.argwhere(~ok)[:5]}"


@pytest.mark.parametrize("M,n_sc", [(6, 40), (20, 40), (6, 1)])
def test_overflowing_weights(lib, M, n_sc):
    """Weights of 1e306 (finite, so accepted): numerator and demand overflow to
    infinity, alone and together, so ratios are +inf and NaN. A NaN share is
    not an idle window, it counts as initialised, and its model neither
    receives nor gives. Shares, flags and decisions as the oracle's."""
    tre, device, torch = lib
    import oracle as O
    w = _workload(M, 300, 1, 500, 77, 2, 4)
    h = w.generate(0, 1).trace(0)
    # a request that waits in the first window of model 0 and is admitted there,
    # then the trace a second later
    n = int(np.searchsorted(h["ts"], 149_000))
    head = E._pack([(0, 0, 1 << 20, 0, 0), (400, 0, 1 << 20, 0x81, 500), (450, 0, 1 << 20, 2, 9), (480, 0, 1 << 20, 3, 0)])
    h = {k: np.concatenate([head[k], (v[:n] + 1000) if k == "ts" else v[:n]]) for k, v in h.items()}
    cols, off = P._columns_from_host(torch, [h])
    cfg = dict(w.trace_cfg(), budget=int(np.sum(w.r_init)))  # nothing idle: moves need donors
    ev = tre.tre_load_events(cols["ts"], cols["model"], cols["req"], cols["type"], cols["tokens"], off, cfg)
    pc = {k: np.array(v, copy=True) for k, v in w.profile_columns(1).items()}
    for m, big in ((0, ("w_p", "w_q")), (2, ("w_p",)), (4, ("w_q",)), (3, ("w_p", "w_q"))):  # requests wait for model 3
        for k in big:
            pc[k][m] = 1e306
    pc["r_min"][:] = 0
    prof = tre.pack(pc, tre.PROFILE_DTYPE)
    sc_cols = P._random_scenarios(1, n_sc, 4)
    sc_cols["theta_scale"] = np.random.default_rng(9).uniform(1.0, 60.0, n_sc)
    sc_cols["max_moves"][:] = 8
    sc = tre.pack(sc_cols, tre.SCENARIO_DTYPE)
    tre.tre_check_params(ev, prof, sc)
    o, op = O.get(), O.pack_profiles(pc)
    ref = o.tss_trace(h, cfg["window_ms"], cfg["duration_ms"], op)
    assert np.isnan(ref["S"]).any() and np.isinf(ref["S"]).any()
    g = {k: v.cpu().numpy()[0] for k, v in _eval(tre, ev, prof).items()}
    _same(g["flags"], ref["flags"], "flags")
    _same(g["tss64"], ref["S"], "shares")
    st = tre.stage_outputs(ev)
    tre.tre_eval_stage(ev, prof, st)
    rs = o.stage_tss(ref, cfg["window_ms"], op)
    _same(st["stage64"].cpu().numpy()[0], rs["S"], "stage shares")
    _same(st["flags"].cpu().numpy()[0], rs["flags"], "stage flags")
    cap = ev.n_ticks * 8
    outs = {"rebalance": tre.ctl_outputs(ev, n_sc, cap), "sweep": tre.ctl_outputs(ev, n_sc, cap)}
    tre.tre_rebalance(ev, prof, torch.from_numpy(ref["S"][None].copy()).cuda(), torch.from_numpy(ref["flags"][None].copy()).cuda(),
                      sc, outs["rebalance"])
    tre.tre_sweep(ev, prof, sc, outs["sweep"], torch.empty(tre.tre_workspace_size(ev, n_sc), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    total = 0
    for s in range(n_sc):
        row = np.zeros(1, O.SCENARIO_DTYPE)
        for k in O.SCENARIO_DTYPE.names:
            row[k] = sc_cols[k][s]
        rc = o.control(cfg, op, ref["S"], ref["flags"], row, cap)
        total += int((rc["moves"]["donor"] != 0xFF).sum())
        for how, out in outs.items():
            mv = tre.unpack_moves(out["moves"]).reshape(-1)[s * cap:(s + 1) * cap]
            PT.compare_ctl(mv, int(out["n_moves"][s]), out["r_final"][s].cpu().numpy(), out["r_windows"][s].cpu().numpy(), rc,
                           f"{how} scenario {s}")
    assert total > 0
    ev.close()


def _eval(tre, ev, prof):
    out = tre.tss_outputs(ev, which=("tss64", "flags"))
    tre.tre_eval_tss(ev, prof, out)
    return out


def test_beside_a_capture(lib):
    """A call on a stream of its own while another stream is being captured: the
    capture goes on, and the call's outputs and the graph's are right."""
    tre, device, torch = lib
    w = _workload(8, 200, 4, 250, 21, 4, 8)
    dt = device.upload(w)
    ev = device.load(dt)
    prof = device.profiles(w)
    ref = {k: v.clone() for k, v in _eval(tre, ev, prof).items()}
    got, other = tre.tss_outputs(ev, which=("tss64", "flags")), tre.tss_outputs(ev, which=("tss64", "flags"))
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    x = torch.zeros(1024, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a):
        x.add_(1.0)
        tre.tre_eval_tss(ev, prof, got, stream=b)
        tre.tre_eval_tss(ev, prof, other)
        x.add_(1.0)
    torch.cuda.synchronize()
    for k in ref:
        assert torch.equal(got[k].view(torch.uint8), ref[k].view(torch.uint8)), k
    x.zero_()
    g.replay()
    torch.cuda.synchronize()
    assert float(x.min()) == 2.0 == float(x.max())
    for k in ref:
        assert torch.equal(other[k].view(torch.uint8), ref[k].view(torch.uint8)), k
    ev.close()


def _held(torch):
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_scratch_is_given_back(lib):
    """Scratch of 384 MiB (150 traces x 24 models x 14000 windows, empty): kept past
    the last handle, while the next handles need as much; given back once they
    need less, and by a load that is refused. A call that would need more than
    1 GiB takes none."""
    tre, device, torch = lib
    T, M, nW, big = 150, 24, 14_000, 300 << 20
    cols = {k: torch.zeros(16, dtype=d, device="cuda") for k, d in
            (("ts", torch.int64), ("model", torch.uint8), ("req", torch.uint32), ("type", torch.uint8), ("tokens", torch.uint16))}
    w = _workload(M, nW, T, 100, 1, 50, 100)
    prof = tre.pack(w.profile_columns(T), tre.PROFILE_DTYPE)

    def load(off, cfg, **kw):
        return tre.tre_load_events(cols["ts"], cols["model"], cols["req"], cols["type"], cols["tokens"], off, cfg, **kw)

    def turn(n_traces, n_windows):
        ev = load(np.zeros(n_traces + 1, np.int64), dict(w.trace_cfg(), duration_ms=100 * n_windows))
        t32 = tre.tss_outputs(ev, which=("flags",))
        tre.tre_eval_tss(ev, prof, t32)
        torch.cuda.synchronize()
        assert int(t32["flags"].min()) == 1 == int(t32["flags"].max())  # idle, never initialised
        ev.close()
    turn(1, 1000)
    before = _held(torch)
    turn(T, nW)
    assert _held(torch) > before + big
    turn(T, nW)
    assert _held(torch) > before + big
    turn(1, 1000)
    assert _held(torch) < before + (16 << 20)
    turn(T, 38_000)
    assert _held(torch) < before + (16 << 20)
    turn(T, nW)
    # a load refused at its last check, after tables of 4 bytes for each of 2^27 ids
    cols["ts"].copy_(torch.arange(16))
    cols["req"].copy_(torch.full((16,), 1 << 27, dtype=torch.int64))  # sixteen ARRIVE rows of one id
    with pytest.raises(tre.TreError) as e:
        load(np.array([0, 16]), w.trace_cfg())
    assert e.value.code == tre.TRE_ESTATE
    assert _held(torch) < before + (16 << 20)


def test_streams_and_threads(lib):
    """Calls of several threads on streams of their own, at once, on trace sets of
    their own: each one's outputs are those of the same call alone."""
    import threading
    tre, device, torch = lib
    sets, errors = [], []
    for i, (M, nW, T) in enumerate([(8, 700, 5), (20, 400, 9), (3, 1500, 3), (16, 900, 2)]):
        w = _workload(M, nW, T, 250, 40 + i, 4, 8)
        ev, prof = device.load(device.upload(w)), device.profiles(w)
        ref = {k: v.clone() for k, v in tre.tss_outputs(ev).items()}
        tre.tre_eval_tss(ev, prof, ref)
        st = tre.stage_outputs(ev)
        tre.tre_eval_stage(ev, prof, st)
        sets.append((ev, prof, ref, st))
    torch.cuda.synchronize()

    def work(ev, prof, ref, sref):
        try:
            stream = torch.cuda.Stream()
            for _ in range(12):
                with torch.cuda.stream(stream):
                    outs = [tre.tss_outputs(ev) for _ in range(3)]
                    st = tre.stage_outputs(ev)
                    for o in outs:
                        tre.tre_eval_tss(ev, prof, o)
                    tre.tre_eval_stage(ev, prof, st)
                stream.synchronize()
                for o in outs:
                    for k in ref:
                        assert torch.equal(o[k].view(torch.uint8), ref[k].view(torch.uint8)), k
                for k in sref:
                    assert torch.equal(st[k].view(torch.uint8), sref[k].view(torch.uint8)), k
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(e)
    threads = [threading.Thread(target=work, args=s) for s in sets]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors, errors
    for s in sets:
        s[0].close()
