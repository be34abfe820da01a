"""Waits of the 2D sweeps kept on the chip (stride_sweep_wait)."""
import threading

import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2110_03345_amd as S
    from paper_2110_03345_amd import _abi


@pytest.fixture(autouse=True)
def defaults():
    yield
    _abi.stride_sweep_wait(-1)
    _abi.stride_check_finite(True)
    _abi.stride_timing_enable(False)


class Shot:
    """A shot with its inputs on the device."""

    def __init__(self, shape=(150, 141), nt=60, nrec=12, seed=0, **kw):
        self.w = W.tiny_2d(n=shape, nt=nt, nrec=nrec, seed=seed, **kw)
        self.plan = S.Plan.from_workload(self.w)
        self.vp = torch.from_numpy(self.w.vp).cuda()
        self.wav = torch.from_numpy(self.w.wavelet).cuda()
        g = torch.Generator(device="cuda").manual_seed(seed)
        self.data = torch.randn((nrec, nt), device="cuda", generator=g)

    def forward(self):
        return self.plan.forward(self.vp, self.wav)

    def gradient(self, ws=None):
        """traces, misfit, dvp"""
        tr = torch.empty_like(self.data)
        m, d = self.plan.gradient(self.vp, self.wav, self.data, ws=ws, traces=tr)
        return tr, m, d

    def autograd(self, ws):
        """traces, dvp, dwavelet of forward_save and backward"""
        tr = self.plan.forward_save(self.vp, self.wav, ws)
        d, dw = self.plan.backward(self.vp, self.wav, self.data, ws, want_dwavelet=True)
        return tr, d, dw


def launches(f):
    """(forward steps, forward launches, adjoint steps, adjoint launches) of f()"""
    _abi.stride_timing_enable(True)
    f()
    _, fs, fl, _, as_, al = _abi.stride_timing_read()
    _abi.stride_timing_enable(False)
    return fs, fl, as_, al


def test_a_thread_can_choose_single_steps():
    """0 polls: a launch per step, the same bits; other threads keep their sweeps."""
    x = Shot()
    ref = x.gradient()
    assert launches(x.gradient) == (59, 1, 60, 1)
    _abi.stride_sweep_wait(0)
    assert launches(x.gradient) == (59, 59, 60, 60)
    assert all(torch.equal(a, b) for a, b in zip(x.gradient(), ref))
    other = []
    t = threading.Thread(target=lambda: other.append(launches(x.forward)))
    t.start()
    t.join()
    assert other == [(59, 1, 0, 0)]
    _abi.stride_sweep_wait(-1)
    assert launches(x.gradient) == (59, 1, 60, 1)


# two steps per exchange; one, with one quad per thread; one, with two
GIVE_UP = [dict(), dict(space_order=10), dict(shape=(1010, 1037), nt=24)]


@pytest.mark.parametrize("kw", GIVE_UP, ids=["two_steps", "one_quad", "two_quads"])
def test_blocks_that_give_up_leave_together(kw):
    """A bound of one poll, which blocks reach at once: every wave of a block leaves
    in the same step, the call reports it and the outputs are NaN; the same plan
    and workspace then solve again."""
    x = Shot(**kw)
    ws = x.plan.workspace(S.STRIDE_MODE_GRADIENT)
    ref = x.gradient(ws)
    for _ in range(3):
        _abi.stride_sweep_wait(1)
        with pytest.raises(S.StrideError) as e:
            x.forward()
        assert e.value.code == _abi.STRIDE_E_HIP
        out = [torch.zeros_like(t) for t in ref]
        with pytest.raises(S.StrideError) as e:
            _abi.stride_plan_gradient(x.plan.handle, x.vp, x.wav, x.data, *out, ws)
        assert e.value.code == _abi.STRIDE_E_HIP
        assert all(t.isnan().all() for t in out)
        _abi.stride_check_finite(False)
        assert x.forward().isnan().all()
        _abi.stride_check_finite(True)
        _abi.stride_sweep_wait(-1)
        assert all(torch.equal(a, b) for a, b in zip(x.gradient(ws), ref))


@pytest.mark.parametrize("stopped", ["forward", "backward"])
def test_every_output_of_a_stopped_sweep_is_nan(stopped):
    """With the finite check off the NaN outputs are the only sign: the model and
    the wavelet gradient, when the adjoint's sweep stopped and when the forward's
    did, the adjoint then running as single steps."""
    x = Shot()
    ws = x.plan.workspace(S.STRIDE_MODE_GRADIENT)
    _abi.stride_check_finite(False)
    _abi.stride_sweep_wait(1 if stopped == "forward" else -1)
    tr = x.plan.forward_save(x.vp, x.wav, ws)
    assert bool(tr.isnan().all()) == (stopped == "forward")
    _abi.stride_sweep_wait(0 if stopped == "forward" else 1)
    dvp, dwav = torch.zeros_like(x.vp), torch.zeros_like(x.wav)
    _abi.stride_backward(x.plan.handle, x.vp, x.wav, x.data, dvp, dwav, ws)
    assert dvp.isnan().all() and dwav.isnan().all()


def _run(eng, stream, chunks):
    """Runs the engine to its end, chunk k with the bound chunks[k] (the last one on)."""
    k, done = 0, []
    while True:
        _abi.stride_sweep_wait(chunks[min(k, len(chunks) - 1)])
        n, fin = _abi.stride_engine_run(eng, 16, 4, stream)
        done += fin
        k += 1
        if n == 0:
            stream.synchronize()
            return done


def _attach(eng, x, mode, stream):
    out = [torch.zeros_like(x.data), torch.zeros(1, dtype=torch.float64, device="cuda"),
           torch.zeros_like(x.vp)]
    ws = x.plan.workspace(mode)
    torch.cuda.synchronize()
    _abi.stride_engine_attach(eng, x.plan.handle, mode, x.vp, float(x.w.vp.max()), x.wav, x.data, *out,
                              ws, stream)
    return (out if mode == S.STRIDE_MODE_GRADIENT else out[:1]), ws


def test_engine_tells_of_stopped_sweeps_and_goes_on():
    """A stopped sweep, in the last chunk as in an earlier one, makes the outputs of
    its own shot NaN and no other's, and is told once; then the engine's shots
    sweep again."""
    x, y = Shot(seed=1), Shot(seed=2)
    grad, fwd = S.STRIDE_MODE_GRADIENT, S.STRIDE_MODE_FORWARD
    ref = {(id(a), grad): a.gradient() for a in (x, y)}
    ref.update({(id(a), fwd): (a.forward(),) for a in (x, y)})
    eng = _abi.stride_engine_create(S.make_grid(**x.w.grid_kwargs()), 4, 16, 16, False)
    stream = torch.cuda.Stream()
    try:
        for mode, bad in ((fwd, [-1, -1, -1, 1]), (grad, [1, -1]), (grad, [-1] * 7 + [1]), (grad, [1])):
            # x meets the bounds of `bad`; y comes in its last chunks or after them
            out, ws = _attach(eng, x, mode, stream)
            for k in range(len(bad)):
                _abi.stride_sweep_wait(bad[k])
                _abi.stride_engine_run(eng, 16, 4, stream)
            other, wy = _attach(eng, y, mode, stream)
            _run(eng, stream, [-1])
            assert all(t.isnan().all() for t in out), (mode, bad)
            assert all(torch.equal(a, b) for a, b in zip(other, ref[id(y), mode])), (mode, bad)
            with pytest.raises(S.StrideError) as e:
                _abi.stride_engine_check(eng)
            assert e.value.code == _abi.STRIDE_E_HIP
            _abi.stride_engine_check(eng)
            for slot in (0, 1):
                _abi.stride_engine_detach(eng, slot)
            out, ws = _attach(eng, x, mode, stream)
            _run(eng, stream, [-1])
            _abi.stride_engine_check(eng)
            assert all(torch.equal(a, b) for a, b in zip(out, ref[id(x), mode]))
            _abi.stride_engine_detach(eng, 0)
    finally:
        _abi.stride_engine_destroy(eng)


def test_inversion_and_server_refuse_stopped_sweeps():
    """Their callers get an error, not NaN gradients (of which a descent step would
    make a model at its lower bound)."""
    from paper_2110_03345_amd import fwi
    from paper_2110_03345_amd.serving import Server
    from workloads.serving_mix import materialise, request_stream
    x = Shot(nrec=12)
    w = x.w
    sv = fwi.Survey(w.shape, w.spacing, w.space_order, w.nb, w.vref, w.dt, w.nt, w.src_xyz, w.rec_xyz,
                    x.wav[0], x.data.expand(2, -1, -1).contiguous())
    batch = fwi.BatchGradient(sv, 2)
    try:
        ref = batch(x.vp, sv.wavelet, sv.observed, [0, 1])
        _abi.stride_sweep_wait(1)
        with pytest.raises(S.StrideError) as e:
            batch(x.vp, sv.wavelet, sv.observed, [0, 1])
        assert e.value.code == _abi.STRIDE_E_HIP
        _abi.stride_sweep_wait(-1)
        J, g = batch(x.vp, sv.wavelet, sv.observed, [0, 1])
        assert J == ref[0] and torch.equal(g, ref[1])
    finally:
        batch.close()
    specs = [materialise(s, nrec_2d=24, nrec_3d=32)
             for s in request_stream(3, 5, rate_hz=200.0, nt_range=(60, 90), shots_range=(1, 2),
                                     classes_2d=(150,), classes_3d=())]
    srv = Server(hbm_budget=1 << 30, max_slots=4, max_chunk=16)
    try:
        _abi.stride_sweep_wait(1)
        with pytest.raises(S.StrideError) as e:
            srv.run(specs, realtime=False)
        assert e.value.code == _abi.STRIDE_E_HIP
        torch.cuda.synchronize()
    finally:
        srv.close()


def test_captured_backward_launches_every_step():
    """stride_backward, the one call that waits for nothing with the finite check off,
    captured: a kernel node per adjoint step and no cooperative launch, and right on
    every replay."""
    import ctypes
    x = Shot()
    ws = x.plan.workspace(S.STRIDE_MODE_GRADIENT)
    _, dref, wref = x.autograd(ws)
    dvp, dwav = torch.empty_like(dref), torch.empty_like(wref)
    _abi.stride_check_finite(False)
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        _abi.stride_backward(x.plan.handle, x.vp, x.wav, x.data, dvp, dwav, ws)
    n = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value > x.w.nt
    g.instantiate()
    for k in range(4):
        dvp.fill_(float(k))
        dwav.zero_()
        x.forward()         # eager work, with a sweep of its own, between the replays
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dvp, dref) and torch.equal(dwav, wref), k


@pytest.mark.parametrize("nt,want", [(2, (1, 1, 2, 2)), (9, (8, 8, 9, 9)), (10, (9, 9, 10, 1)),
                                     (11, (10, 1, 11, 1))])
def test_short_sweeps_launch_every_step(nt, want):
    """Sweeps of fewer than ten steps, which a cooperative launch would slow down."""
    x = Shot(nt=nt)
    assert launches(x.gradient) == want
    assert launches(x.forward) == want[:2] + (0, 0)


@pytest.mark.parametrize("kw", [dict(shape=(50, 41)), *GIVE_UP], ids=["one_tile", "two_steps", "one_quad", "two_quads"])
@pytest.mark.parametrize("frac", [1.0, 0.7, 0.5])
def test_histories_run_as_sweeps(kw, frac):
    """Full history: one launch forward and one adjoint.  Segmented: the forward in a
    launch up to each stored start, the last two segments in one, a launch to
    recompute each segment but the last, and one adjoint launch a segment.  The
    binomial schedule launches every step.  The same bits throughout."""
    x = Shot(**dict(kw, nt=60))
    ref = x.gradient()
    ws = x.plan.workspace(S.STRIDE_MODE_GRADIENT,
                          int(x.plan.workspace_bytes(S.STRIDE_MODE_GRADIENT) * frac))
    path, steps, K = x.plan.gradient_path(ws.numel())
    assert path == (S.STRIDE_PATH_FULL_HISTORY if frac == 1.0 else S.STRIDE_PATH_SEGMENTED)
    want = (59, 1, 60, 1) if frac == 1.0 else (steps, 2 * (K - 1), 60, K)
    assert launches(lambda: x.gradient(ws)) == want
    assert all(torch.equal(a, b) for a, b in zip(x.gradient(ws), ref))
    if frac == 0.5:
        x.plan = S.Plan.from_workload(x.w, checkpointing=1)
        assert x.plan.gradient_path(ws.numel())[0] == S.STRIDE_PATH_BINOMIAL
        fs, fl, as_, al = launches(lambda: x.gradient(ws))
        assert fs == fl >= 59 and as_ == al == 60
        assert all(torch.equal(a, b) for a, b in zip(x.gradient(ws), ref))


def test_sweeps_beside_other_work():
    """Threads with a stream each: sweeps of one tile, of many and of two quads a
    thread, and 3D steps that fill the GPU: the bits of each alone."""
    shots = [Shot(shape=(50, 41), nt=300), Shot(nt=200), Shot(shape=(400, 390), nt=120, space_order=10),
             Shot(shape=(1010, 1037), nt=60)]
    w3 = W.tiny_3d(n=(140, 150, 130), nt=40)
    p3 = S.Plan.from_workload(w3)
    vp3, wav3 = torch.from_numpy(w3.vp).cuda(), torch.from_numpy(w3.wavelet).cuda()
    jobs = [x.gradient for x in shots] + [lambda: (p3.forward(vp3, wav3),)]
    refs = [f() for f in jobs]
    torch.cuda.synchronize()
    wrong, gate = [], threading.Barrier(len(jobs))

    def work(f, ref):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                gate.wait()
                for k in range(12):
                    out = f()
                    s.synchronize()
                    if not all(torch.equal(a, b) for a, b in zip(out, ref)):
                        wrong.append(("bits", k))
        except Exception as e:      # (an assertion in a thread is not the test's)
            wrong.append(repr(e))
    threads = [threading.Thread(target=work, args=jr) for jr in zip(jobs, refs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


@pytest.mark.parametrize("chunk,sweeps", [(8, False), (64, True)])
def test_engine_takes_the_cheaper_of_sweeps_and_ticks(chunk, sweeps):
    """Eight shots of a grid of which the chip holds one sweep: short chunks tick, all
    shots in one launch, long ones sweep shot after shot.  (A bound of one poll tells
    them apart.)"""
    shots = [Shot(shape=(1010, 1037), nt=65, seed=i) for i in range(8)]
    ref = [x.forward() for x in shots]
    eng = _abi.stride_engine_create(S.make_grid(**shots[0].w.grid_kwargs()), 8, 16, chunk, True)
    stream = torch.cuda.Stream()
    try:
        for bound in (-1, 1):
            out = [_attach(eng, x, S.STRIDE_MODE_FORWARD, stream) for x in shots]
            _abi.stride_sweep_wait(bound)
            while _abi.stride_engine_run(eng, chunk, 8, stream)[0]:
                pass
            stream.synchronize()
            if sweeps and bound == 1:
                with pytest.raises(S.StrideError):
                    _abi.stride_engine_check(eng)
            else:
                _abi.stride_engine_check(eng)
                assert all(torch.equal(o[0], r) for (o, _), r in zip(out, ref))
            for slot in range(8):
                _abi.stride_engine_detach(eng, slot)
    finally:
        _abi.stride_engine_destroy(eng)


def test_autograd_backward_keeps_the_forwards_choice():
    """torch runs backward on a thread of its own, which has made no choice."""
    from paper_2110_03345_amd.autograd import wave_traces
    x = Shot()
    grads = []
    for polls, want in ((-1, (60, 1)), (0, (60, 60)), (-1, (60, 1))):
        _abi.stride_sweep_wait(polls)
        vp = x.vp.clone().requires_grad_()
        seen = []
        traces = wave_traces(vp, x.wav, x.plan)
        # hooks on the backward's thread, before and after it
        traces.register_hook(lambda g: _abi.stride_timing_enable(True))

        def after(g):
            seen.append(_abi.stride_timing_read()[4:])
            _abi.stride_timing_enable(False)
        vp.register_hook(after)
        _abi.stride_sweep_wait(-1)
        (traces * x.data).sum().backward()
        torch.cuda.synchronize()
        assert seen == [want], (polls, seen)
        grads.append(vp.grad)
    assert torch.equal(grads[0], grads[1]) and torch.equal(grads[0], grads[2])
