"""GPU parity of the line solver at the edges of its chunk lengths (8, 16, 24,
32 levels) and register budgets (512, 768, 1024 threads), with tiles that make
one round of workgroups and with tiles that make several, and of the streaming
step on wide grids of few levels.

Tolerances: those of the step and adjoint tests (the chunk length only changes
the order of the double recurrences, whose factors are at most 1 in size).
"""
import pytest

from tests import test_gpu_stream as S
from tests.test_gpu_face4 import Case4, _adjoint_vs_oracle, _steps
from tests.test_gpu_parity import FP32_TOL, FP64_TOL
from tests.test_gpu_walls import WallCase

pytestmark = pytest.mark.gpu
PERIODIC = (False, False)

# (ny, nz): 12 rows fit one round of tiles (chunks of 8, 16, 24 and 32 from nz =
# 1, 65, 129, 193), 520 rows make more than 256 tiles (8, 16, 24 or 32, 32, 24
# and 32 from nz = 1, 33, 65, 97, 129 or 161, 193)
SIZES = [(12, 9), (12, 64), (12, 65), (12, 129), (12, 192), (12, 193), (12, 257), (12, 385),
         (520, 8), (520, 32), (520, 33), (520, 65), (520, 97), (520, 161), (520, 193)]


class PlainCase(WallCase):
    """Uniform x and y, the plain method, on the line solver."""

    def __init__(self, nc, **kw):
        super().__init__(nc, (1, 1, 1), PERIODIC, **kw)
        import oracle as O
        from paper_1805_03426_amd import inputs
        self.yf = inputs.uniform_faces(self.g.y.n)
        self.g = O.Grid(self.xf, self.yf, self.zf, self.m)

    def ctx(self):
        from paper_1805_03426_amd.context import Context
        return Context(self.xf, self.yf, self.zf, self.m, self.ra, self.pr, self.dt, n_avg=self.n_avg,
                       precision=self.precision, step_method="line")


def _case(kind, ny, nz, prec):
    kw = dict(precision=prec, n_avg=3, dt=1e-4 if ny > 100 else 1e-3)
    if kind == "plain":
        return PlainCase((3, ny, nz), **kw)
    return Case4((3, ny, nz), (1, 1, 1), (True, True), z_explicit=0.5, **kw)


@pytest.mark.parametrize("ny,nz", SIZES)
@pytest.mark.parametrize("kind", ["plain", "full"])
def test_steps_at_chunk_edges(kind, ny, nz):
    for prec, tol in (("fp64", FP64_TOL), ("fp32", FP32_TOL)):
        print("case line chunks", kind, ny, nz, prec, flush=True)
        _steps(_case(kind, ny, nz, prec), 3, tol)


@pytest.mark.parametrize("ny,nz", [(12, 9), (12, 65), (12, 130), (12, 257), (520, 8), (520, 34), (520, 66)])
@pytest.mark.parametrize("kind", ["plain", "full"])
def test_adjoint_at_chunk_edges(kind, ny, nz):
    print("case line chunks adjoint", kind, ny, nz, flush=True)
    _adjoint_vs_oracle(_case(kind, ny, nz, "fp64"), 4)


@pytest.mark.parametrize("nx,ny,nz,r", [(258, 130, 1, 0.05), (66, 400, 3, 0.3), (130, 120, 8, 0.9)])
def test_streaming_on_wide_grids_of_few_levels(nx, ny, nz, r):
    """More than one round of line-solver tiles: the streaming step, with
    look-aheads longer than the column."""
    S.test_stream_steps_fp64(nx, ny, nz, r)
    S.test_stream_reverse_steps_fp64(nx, ny, nz, r)


@pytest.mark.parametrize("nx,ny,nz,r", [(64, 20, 130, 0.3), (63, 9, 300, 0.05), (5, 3, 640, 0.9), (180, 170, 90, 0.05)])
def test_streaming_fp32_on_tall_and_middle_grids(nx, ny, nz, r):
    """FP32 columns of more than 128 levels in one round of tiles, and several
    rounds below 4.5e6 cells."""
    S.test_stream_fp32_matches_line_solver_and_sweeps(nx, ny, nz, r, "line")
