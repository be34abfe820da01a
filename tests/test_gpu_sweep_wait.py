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
