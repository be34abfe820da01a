"""The layer's correction where its quads and ranges end, against the oracle's
PML forward: layers that end inside a quad, rows of every remainder by four,
physical extents smaller than a quad or than the stencil, single planes and rows
left over from groups of four.

Tolerance 1e-4 of the norm: FP32 rounding over n steps is a small multiple of
n eps, 120 x 6e-8 x 10 = 7e-5; a wrong neighbour, depth or mask is of order one.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import check_traces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2110_03345_amd as S

CASES = [((40, 3), 7, 8), ((5, 62), 6, 10), ((33, 43), 9, 10), ((2, 2), 10, 8),
         ((9, 7, 3), 6, 8), ((3, 26, 18), 5, 10), ((17, 5, 39), 7, 10), ((12, 13, 64), 4, 8)]


@pytest.mark.parametrize("shape,nb,order", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_pml_edges(shape, nb, order):
    make = W.tiny_2d if len(shape) == 2 else W.tiny_3d
    w = make(n=shape, nt=120, space_order=order, nb=nb, seed=sum(shape))
    rng = np.random.default_rng(nb)
    w.wavelet = rng.standard_normal(w.wavelet.shape).astype(np.float32)
    ref = oracle.forward_pml(oracle.Grid(**w.grid_kwargs()), w.vp, w.src_xyz, w.wavelet, w.rec_xyz)
    plan = S.Plan.from_workload(w, boundary=1)
    tr = plan.forward(torch.from_numpy(w.vp).cuda(), torch.from_numpy(w.wavelet).cuda())
    check_traces(tr.cpu().numpy(), ref, 1e-4)


@pytest.mark.parametrize("order", [8, 10])
def test_pml_beyond_the_cache(order):
    """A grid whose layer writes past the Infinity Cache (non-temporal stores), with
    sources and receivers at corners of the physical grid and a layer of a thousand
    times the usual strength, so that in a few steps it changes the traces by a
    twelfth to a quarter."""
    shape, nt = (171, 150, 163), 26
    w = W.tiny_3d(n=shape, nt=nt, space_order=order, nb=30, nsrc=4, nrec=40, seed=order, vref=1.5e6)
    rng = np.random.default_rng(order)
    ext = np.array([(n - 1) * w.spacing for n in shape])
    # four corners; a source and ten receivers within two cells of each
    edge = np.repeat(rng.integers(0, 2, (4, 3)), 11, axis=0) * ext
    points = edge + np.where(edge > 0, -1, 1) * rng.uniform(0, 2, (44, 3)) * w.spacing
    w.src_xyz, w.rec_xyz = points[::11], np.delete(points, np.s_[::11], axis=0)
    w.wavelet = rng.standard_normal((4, nt)).astype(np.float32)
    ref = oracle.forward_pml(oracle.Grid(**w.grid_kwargs()), w.vp, w.src_xyz, w.wavelet, w.rec_xyz)
    plan = S.Plan.from_workload(w, boundary=1)
    tr = plan.forward(torch.from_numpy(w.vp).cuda(), torch.from_numpy(w.wavelet).cuda()).cpu().numpy()
    check_traces(tr, ref, 1e-4)
