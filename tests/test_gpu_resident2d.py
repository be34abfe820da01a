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
