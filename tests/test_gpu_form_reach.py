"""Tests of one form of the step that make sure that this form runs: the streaming
step at the edges of its tiles, blocks, copies and look-aheads (columns beyond the
line solver stream at every size, flat grids of many tiles with few levels), its
variants, the NaN canaries of both, with 16-byte copies and with 4-byte ones chosen
by the fields' alignment, and the column sweeps on columns beyond the line solver.
References and tolerances: those of the tests that the checks come from."""
import pytest
import torch

import oracle as O
from paper_1805_03426_amd import inputs
from tests import test_gpu_stream as S
from tests.test_gpu_canary import _run
from tests.test_gpu_face4 import Case4, _steps
from tests.test_gpu_parity import FP32_TOL, FP64_TOL, Case, host, rel_max
from tests.test_gpu_walls import WallCase

pytestmark = pytest.mark.gpu
CALLS = ("scalar_step", "scalar_steps", "scalar_step_backward", "scalar_steps_backward")


def _streams(ctx, calls=CALLS):
    for call in calls:
        assert ctx.step_form(call) == "stream", call


# r = 0.05, 0.3, 0.9, 2: one size for each compiled look-ahead; N_x odd: copies of 4 bytes
TALL = [(2, 1, 641, 0.05), (2, 2, 643, 0.3), (64, 4, 648, 0.05), (66, 5, 647, 0.9), (62, 3, 649, 0.3), (130, 9, 644, 0.05),
        (258, 13, 641, 0.05), (192, 8, 642, 2.0), (65, 6, 650, 0.9), (1, 1, 645, 2.0), (127, 5, 656, 0.05)]
FLAT = [(1030, 516, 7, 0.05), (1026, 514, 8, 0.3), (1026, 510, 9, 0.9), (1025, 513, 9, 0.05)]


@pytest.mark.parametrize("nx,ny,nz,r", TALL + FLAT)
def test_streaming_edges_fp64(nx, ny, nz, r):
    faces, dt, _, _ = S._case(nx, ny, 1, r)
    with S._ctx((faces[0], faces[1], S._faces(nx, ny, nz, r)[2]), dt, "fp64") as ctx:
        _streams(ctx)
    S.test_stream_steps_fp64(nx, ny, nz, r)
    S.test_stream_reverse_steps_fp64(nx, ny, nz, r)


@pytest.mark.parametrize("nx,ny,nz,r", TALL)
def test_streaming_edges_fp32(nx, ny, nz, r):
    faces, dt, _, _ = S._case(nx, ny, 1, r)
    with S._ctx((faces[0], faces[1], S._faces(nx, ny, nz, r)[2]), dt, "fp32") as ctx:
        _streams(ctx)
    S.test_stream_fp32_matches_line_solver_and_sweeps(nx, ny, nz, r, "sweep")


VARIANTS = [(4, (False, False), 0.0), (4, (True, True), 0.5), (2, (True, True), 0.0), (2, (False, False), 0.5),
            (2, (True, False), 0.5)]


class _Variant(WallCase):
    """Second order on uniform x and y."""

    def __init__(self, nc, walls, wz, m=(1, 1, 1), **kw):
        super().__init__(nc, m, walls, **kw)
        import dataclasses
        self.yf = inputs.uniform_faces(self.g.y.n)
        self.g = O.Grid(self.xf, self.yf, self.zf, self.m, periodic=(not walls[0], not walls[1], False))
        self.z_explicit = wz
        self.p = dataclasses.replace(self.p, z_explicit=wz)

    def ctx(self):
        from paper_1805_03426_amd.context import Context
        side = ["walls" if w else "periodic" for w in self.walls]
        return Context(self.xf, self.yf, self.zf, self.m, self.ra, self.pr, self.dt, n_avg=self.n_avg,
                       precision=self.precision, side_x=side[0], side_y=side[1], z_explicit=self.z_explicit)


def _variant(order, nc, walls, wz, **kw):
    return Case4(nc, (1, 1, 1), walls, z_explicit=wz, **kw) if order == 4 else _Variant(nc, walls, wz, **kw)


@pytest.mark.parametrize("nc", [(2, 2, 520), (4, 3, 400), (66, 5, 321), (34, 9, 500), (130, 6, 640)])
@pytest.mark.parametrize("order,walls,wz", VARIANTS)
def test_streaming_variants(order, walls, wz, nc):
    for prec, tol in (("fp64", FP64_TOL), ("fp32", FP32_TOL)):
        print("case form reach variant", order, walls, wz, nc, prec, flush=True)
        c = _variant(order, nc, walls, wz, precision=prec, dt=2e-6, n_avg=3)   # (short look-aheads)
        with c.ctx() as ctx:
            _streams(ctx, CALLS[:2])
        _steps(c, 4, tol)


@pytest.mark.parametrize("offset", [64, 1])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("order,walls,wz", VARIANTS)
def test_canaries_streaming_variants(order, walls, wz, prec, offset):
    print("case canaries streaming variants", order, walls, wz, prec, offset, flush=True)
    kw = dict(precision=prec, n_avg=3, dt=2e-6)   # (short look-aheads)
    nc, m = (35, 5, 160), (2, 2, 2)   # 70 x 10 x 320
    c = Case4(nc, m, walls, z_explicit=wz, **kw) if order == 4 else _Variant(nc, walls, wz, m=m, **kw)
    c.th0 = inputs.theta_initial(c.zf, c.g.x.n, c.g.y.n, noise=0.1, seed=2)
    c.U, c.V, c.W = c.coarse_velocity()
    c.U, c.V = c.to_lib(c.U, c.V)
    with c.ctx() as ctx:
        _streams(ctx, CALLS[:2])
        _run(c, ctx, offset)


@pytest.mark.parametrize("offset", [64, 1])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("method", ["auto", "sweep"])
def test_canaries_tall(method, prec, offset):
    """700 levels: streaming steps and reverse steps, or the column sweeps."""
    print("case canaries tall", method, prec, offset, flush=True)
    c = Case((32, 4, 350), (2, 2, 2), 2.0, kmax=1, n_avg=3, precision=prec, dt=1e-5)
    with c.ctx(method) as ctx:
        for call in CALLS:
            assert ctx.step_form(call) == ("stream" if method == "auto" else "sweep")
        _run(c, ctx, offset)


@pytest.mark.parametrize("nz,ckpt", [(700, 2), (1024, 3)])
def test_tall_sweeps_adjoint_fp64(nz, ckpt):
    """The checkpointed rollout's gradients on columns beyond the line solver with
    the seed solve, the reverse steps and the start-up step's reverse as column
    sweeps, against the oracle's discrete adjoint (5 steps)."""
    print("case tall sweeps adjoint", nz, flush=True)
    from paper_1805_03426_amd.autograd import rollout
    case = Case((3, 5, nz // 2), (3, 1, 2), 2.0, kmax=1, n_avg=3, ra=1e4, dt=2e-4)
    target = inputs.theta_initial(case.zf, case.g.x.n, case.g.y.n, seed=3)
    _, w0, wU, wV, wW = O.rollout_loss_grad(case.g, case.p, case.th0, case.U, case.V, case.W, 5, target)
    with case.ctx("sweep") as ctx:
        for call in CALLS:
            assert ctx.step_form(call) == "sweep"
        th = case.d(case.th0).requires_grad_(True)
        U, V, W = (case.d(a).requires_grad_(True) for a in (case.U, case.V, case.W))
        out = rollout(ctx, th, U, V, W, 5, ckpt)
        torch.autograd.backward(out, out.detach() - case.d(target))
        got = [host(t.grad) for t in (th, U, V, W)]
    for a, b in zip(got, (w0, wU, wV, wW)):
        assert rel_max(a, b) <= 1e-11
