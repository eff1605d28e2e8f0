"""GPU parity of the streaming forward step's variants (side walls, fourth-order
faces, explicit z share): columns of more than 128 levels in one round of tiles
and grids of 2.5e6 cells and more stream.  Axes shorter than the stencil, ragged
tiles, both copy widths, one and several z segments, every look-ahead (r = tau
kappa / h^2 grows with dt) and one past them all (the line solver), every step
type, against the oracle at the tolerances of the other step tests; wall faces
that hold NaN are not read."""
import numpy as np
import pytest

import oracle as O
from paper_1805_03426_amd import inputs
from tests.test_gpu_face4 import Case4, _steps
from tests.test_gpu_parity import FP32_TOL, FP64_TOL, host, rel_max
from tests.test_gpu_zweight import ZCase

pytestmark = pytest.mark.gpu
PERIODIC = (False, False)


class UniformZ(ZCase):
    """ZCase on uniform y (second-order faces)."""

    def __init__(self, nc, walls, z_explicit, **kw):
        super().__init__(nc, (1, 1, 1), walls, z_explicit, **kw)
        self.yf = inputs.uniform_faces(self.g.y.n)
        self.g = O.Grid(self.xf, self.yf, self.zf, self.m, periodic=(not walls[0], not walls[1], False))


def _case(order, nc, walls, wz, **kw):
    if order == 4:
        return Case4(nc, (1, 1, 1), walls, z_explicit=wz, **kw)
    return UniformZ(nc, walls, wz, **kw)


VARIANTS = [(4, PERIODIC, 0.0), (4, (True, True), 0.5), (2, (True, False), 0.0), (2, (False, True), 0.5),
            (2, PERIODIC, 0.3), (4, (False, True), 0.0)]


@pytest.mark.parametrize("nc,dt", [
    ((1, 1, 130), 1e-3), ((2, 2, 129), 1e-3), ((4, 3, 200), 1e-3), ((66, 5, 150), 1e-4), ((130, 6, 333), 1e-4),
    ((8, 9, 300), 6e-4), ((6, 5, 400), 8e-4), ((4, 4, 300), 3e-3), ((4, 4, 300), 2e-2), ((6, 3, 640), 2e-4),
    ((33, 6, 140), 1e-4),
])
@pytest.mark.parametrize("order,walls,wz", VARIANTS)
def test_stream_variant_steps(order, walls, wz, nc, dt):
    for prec, tol in (("fp64", FP64_TOL), ("fp32", FP32_TOL)):
        print("case stream variant", order, walls, wz, nc, dt, prec, flush=True)
        if walls != PERIODIC and min(nc[:2]) < 2:
            continue
        _steps(_case(order, nc, walls, wz, precision=prec, dt=dt, n_avg=3), 4, tol)


@pytest.mark.parametrize("nc", [(194, 132, 98), (135, 190, 180), (1280, 500, 4)])
@pytest.mark.parametrize("order,walls,wz", [(4, (True, True), 0.5), (2, (True, True), 0.0)])
def test_stream_variant_steps_large(order, walls, wz, nc):
    """Several rounds of tiles, 16-byte and 4-byte copies, fewer levels than a block."""
    for prec, tol in (("fp64", FP64_TOL), ("fp32", FP32_TOL)):
        print("case stream variant large", order, walls, wz, nc, prec, flush=True)
        _steps(_case(order, nc, walls, wz, precision=prec, dt=2e-5, n_avg=3), 2, tol)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_stream_variant_ignores_wall_faces(prec):
    """The velocity on wall faces is taken as zero whatever the arrays hold."""
    print("case stream variant wall faces", prec, flush=True)
    c = _case(4, (12, 10, 150), (True, True), 0.5, precision=prec, dt=1e-3, n_avg=3)
    u, v, w = c.dense_velocity()
    ul, vl = c.to_lib(u, v)
    ul, vl = ul.copy(), vl.copy()
    ul[:, :, 0] = np.nan
    vl[:, 0] = np.nan
    th = inputs.theta_initial(c.zf, c.g.x.n, c.g.y.n, noise=0.1, seed=2)
    with c.ctx() as ctx:
        out = ctx.empty(ctx.shape_cell)
        ctx.scalar_step(1, c.d(0.9 * th), c.d(th), out, c.d(ul), c.d(vl), c.d(w))
        got = host(out)
    assert rel_max(got, O.scalar_step(c.g, c.p, 1, 0.9 * th, th, u, v, w)) <= (FP64_TOL if prec == "fp64" else FP32_TOL)
