"""3D step kernels where their vectors, tiles and chunks end, against the FP64
oracle: rows that end inside a vector of four or two points, in the tile and in
its halo; grids a few points past a tile (64 x 16 and 64 x 8) or a chunk of
planes (4 to 16); every launch mode (leapfrog, stored v, imaging in pairs, fused
adjoint, fourth-order launches, both medium steps).

Tolerance 1e-4 of the norm (1e-3 of every trace's and 3e-4 of each region's own
norm): the kernels and the oracle differ by FP32 rounding only, whose relative
size after n steps is a small multiple of n eps, 60 x 6e-8 x 10 = 4e-5; a wrong
tap, mask or chunk gives an error of order one where it touches.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from parity import check_field, check_traces

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2110_03345_amd as S

TOL = 1e-4
# padded widths 61 .. 68 (every remainder by four, either side of a tile) and 133;
# rows and planes around the tile heights and chunk lengths
SHAPES = [(11, 12, 51), (12, 9, 52), (13, 23, 53), (9, 24, 54), (27, 25, 55), (24, 7, 57),
          (25, 39, 58), (22, 22, 123)]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def case(shape, order, **kw):
    w = W.tiny_3d(n=shape, nt=60, space_order=order, nb=5, nsrc=3, nrec=24, seed=sum(shape))
    return w, oracle.Grid(**w.grid_kwargs(), **kw)


@pytest.mark.parametrize("order", [8, 10])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_leapfrog_gradient(shape, order):
    w, g = case(shape, order)
    obs = np.zeros((len(w.rec_xyz), w.nt), np.float32)
    ref, J, dref = oracle.gradient(g, w.vp, w.src_xyz, w.wavelet, w.rec_xyz, obs)
    for ckpt in (0, 1):     # stored v; binomial schedule (fused adjoint) in less memory
        plan = S.Plan.from_workload(w, checkpointing=ckpt)
        full = plan.workspace_bytes(S.STRIDE_MODE_GRADIENT)
        ws = plan.workspace(S.STRIDE_MODE_GRADIENT, full if ckpt == 0 else full // 3)
        tr = torch.empty(ref.shape, dtype=torch.float32, device="cuda")
        m, d = plan.gradient(dev(w.vp), dev(w.wavelet), dev(obs), ws=ws, traces=tr)
        check_traces(tr.cpu().numpy(), ref, TOL)
        assert abs(m.item() - J) <= TOL * J
        check_field(d.cpu().numpy(), dref, TOL)


@pytest.mark.parametrize("shape", SHAPES[::2], ids=lambda s: "x".join(map(str, s)))
def test_fourth_order_gradient(shape):
    w, g = case(shape, 10, time_order=4)
    obs = np.zeros((len(w.rec_xyz), w.nt), np.float32)
    ref, J, dref = oracle.gradient(g, w.vp, w.src_xyz, w.wavelet, w.rec_xyz, obs)
    plan = S.Plan.from_workload(w, time_order=4)
    tr = torch.empty(ref.shape, dtype=torch.float32, device="cuda")
    m, d = plan.gradient(dev(w.vp), dev(w.wavelet), dev(obs), traces=tr)
    check_traces(tr.cpu().numpy(), ref, TOL)
    assert abs(m.item() - J) <= TOL * J
    check_field(d.cpu().numpy(), dref, TOL)


@pytest.mark.parametrize("power", [0, 2])
@pytest.mark.parametrize("shape", SHAPES[1::2], ids=lambda s: "x".join(map(str, s)))
def test_medium_gradient(shape, power):
    w, g = case(shape, 10)
    rng = np.random.default_rng(4)
    rho = (1000.0 * (1 + 0.1 * rng.uniform(-1, 1, shape))).astype(np.float32)
    alpha = rng.uniform(0.5, 5.0, shape) / (2 * np.pi * 5e5) ** power
    alpha = alpha.astype(np.float32)
    obs = np.zeros((len(w.rec_xyz), w.nt), np.float32)
    ref, J, dref = oracle.gradient_medium(g, w.vp, w.src_xyz, w.wavelet, w.rec_xyz, obs, rho, alpha,
                                          power)
    plan = S.Plan.from_workload(w)
    tr = torch.empty(ref.shape, dtype=torch.float32, device="cuda")
    m, d = plan.gradient_medium(dev(w.vp), dev(w.wavelet), dev(obs), dev(rho), dev(alpha), power,
                                traces=tr)
    check_traces(tr.cpu().numpy(), ref, TOL)
    assert abs(m.item() - J) <= TOL * J
    check_field(d.cpu().numpy(), dref, TOL)
