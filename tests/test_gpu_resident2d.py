"""2D sweeps kept on the chip, where their tiles, quads and tables end, against
the FP64 oracle: one tile and many, one and two quads per thread (from a million
points on), rows that end inside a quad, two to sixty steps, more sources and
receivers in one tile than its tap tables hold, bilinear and windowed-sinc
points on tile edges, and every workspace (full history, segments, binomial).

Tolerance 1e-4 of the norm: the kernels and the oracle differ by FP32 rounding
only, whose relative size after n steps is a small multiple of n eps, 60 x 6e-8
x 10 = 4e-5; a wrong frame, tap or mask gives an error of order one where it
touches.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import check_field, check_traces, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2110_03345_amd as S
    from paper_2110_03345_amd import _abi

TOL = 1e-4
# interior shape, layer, order, steps, interp; padded widths of every remainder by four
CASES = [((22, 30), 5, 8, 60, 0), ((71, 57), 5, 8, 60, 1), ((139, 246), 6, 10, 60, 0),
         ((260, 213), 5, 10, 31, 1), ((333, 390), 7, 8, 60, 0), ((90, 121), 4, 8, 2, 0),
         ((90, 122), 4, 10, 3, 1), ((401, 77), 3, 8, 24, 0), ((1010, 1037), 12, 8, 40, 0),
         ((1007, 1048), 10, 10, 21, 0)]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()


@pytest.mark.parametrize("shape,nb,order,nt,interp", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_resident_sweeps(shape, nb, order, nt, interp):
    w = W.tiny_2d(n=shape, nt=nt, space_order=order, nb=nb, seed=sum(shape))
    rng = np.random.default_rng(nt)
    ext = np.array([(n - 1) * w.spacing for n in shape])
    # 90 sources in a patch of a few cells, 90 receivers in it, 150 along the diagonal
    patch = 0.45 * ext + rng.uniform(0, 6, (180, 2)) * w.spacing
    line = np.linspace(0.06, 0.94, 150)[:, None] * ext
    w.src_xyz, w.rec_xyz = patch[:90], np.concatenate([patch[90:], line])
    w.wavelet = rng.standard_normal((90, nt)).astype(np.float32)
    gt = rng.standard_normal((240, nt)).astype(np.float32)
    g = oracle.Grid(**w.grid_kwargs(), interp=interp)
    ref = oracle.forward(g, w.vp, w.src_xyz, w.wavelet, w.rec_xyz)
    dref, wref = oracle.adjoint(g, w.vp, w.src_xyz, w.wavelet, w.rec_xyz, gt)
    plan = S.Plan.from_workload(w, interp=interp)
    check_traces(plan.forward(dev(w.vp), dev(w.wavelet)).cpu().numpy(), ref, TOL)
    full = plan.workspace_bytes(S.STRIDE_MODE_GRADIENT)
    # (the smallest grid's traces leave no room for less than 0.6)
    for frac in (1.0,) if nt < 20 else (1.0, 0.6) if shape[0] < 30 else (1.0, 0.6, 0.4):
        ws = plan.workspace(S.STRIDE_MODE_GRADIENT, int(full * frac))
        tr = plan.forward_save(dev(w.vp), dev(w.wavelet), ws)
        dvp, dwav = plan.backward(dev(w.vp), dev(w.wavelet), dev(gt), ws, want_dwavelet=True)
        check_traces(tr.cpu().numpy(), ref, TOL)
        check_field(dvp.cpu().numpy(), dref, TOL)
        assert rel(dwav.cpu().numpy(), wref) < TOL


@pytest.mark.parametrize("shape,nshots", [((70, 85), 14), ((300, 333), 5), ((611, 590), 3)],
                         ids=lambda v: str(v).replace(" ", ""))
@pytest.mark.parametrize("ticks", [[64], [8, 1, 16, 2], [1, 64, 4]], ids=str)
def test_engine_sweeps(shape, nshots, ticks):
    """Slots whose chunks run as sweeps, as ticks and as both, more of them than
    one launch takes: the bits of the single-shot solves."""
    nt, rng = 75, np.random.default_rng(nshots)
    w = W.tiny_2d(n=shape, nt=nt, nb=6, nrec=40)
    eng = _abi.stride_engine_create(S.make_grid(**w.grid_kwargs()), nshots, 64, 64, True)
    stream = torch.cuda.Stream()
    jobs = []
    for i in range(nshots):
        w.src_xyz = rng.uniform(0.2, 0.8, (2, 2)) * [(n - 1) * w.spacing for n in shape]
        plan = S.Plan.from_workload(w)
        vp, wav = dev(w.vp), dev(rng.standard_normal((2, nt)))
        obs, tr = dev(rng.standard_normal((40, nt))), torch.empty((40, nt), device="cuda")
        mis, dvp = torch.zeros(1, dtype=torch.float64, device="cuda"), torch.empty_like(vp)
        mode = S.STRIDE_MODE_FORWARD if i % 3 == 1 else S.STRIDE_MODE_GRADIENT
        ws = plan.workspace(mode)
        torch.cuda.synchronize()
        _abi.stride_engine_attach(eng, plan.handle, mode, vp, float(w.vp.max()), wav, obs, tr, mis,
                                  dvp, ws, stream)
        jobs.append((plan, mode, vp, wav, obs, tr, mis, dvp, ws))
    done, k = 0, 0
    while done < nshots:
        done += len(_abi.stride_engine_run(eng, ticks[k % len(ticks)], nshots, stream)[1])
        k += 1
    stream.synchronize()
    _abi.stride_engine_destroy(eng)
    for plan, mode, vp, wav, obs, tr, mis, dvp, _ in jobs:
        if mode == S.STRIDE_MODE_FORWARD:
            assert torch.equal(plan.forward(vp, wav), tr)
            continue
        t1 = torch.empty_like(tr)
        m1, d1 = plan.gradient(vp, wav, obs, traces=t1)
        assert torch.equal(t1, tr) and torch.equal(m1, mis) and torch.equal(d1, dvp)
