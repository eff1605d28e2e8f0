"""GPU parity of the line solver with 3 to 4 tiles a CU in FP64, whose chunk lengths
follow a rule of their own (two chunks from 33 to 64 levels, 32 levels a chunk from 65
to 96 in second order), at its edges.  Tolerances: those of the step and adjoint
tests."""
import pytest

from tests.test_gpu_face4 import Case4, _adjoint_vs_oracle, _steps
from tests.test_gpu_line_chunks import PERIODIC, PlainCase
from tests.test_gpu_parity import FP64_TOL

pytestmark = pytest.mark.gpu


def _case(kind, nz):
    kw = dict(precision="fp64", n_avg=3, dt=8e-6)
    if kind == "plain":
        return PlainCase((3, 1800, nz), **kw)   # 900 tiles of 32 x 2
    return Case4((3, 1800, nz), (1, 1, 1), (True, True) if kind == "full" else PERIODIC, z_explicit=0.5, **kw)


@pytest.mark.parametrize("nz", [32, 33, 48, 49, 64, 65, 96])
@pytest.mark.parametrize("kind", ["plain", "full"])
def test_steps(kind, nz):
    print("case line resident", kind, nz, flush=True)
    _steps(_case(kind, nz), 3, FP64_TOL)


@pytest.mark.parametrize("nz", [48, 64, 96])
@pytest.mark.parametrize("kind", ["plain", "full"])
def test_adjoint(kind, nz):
    print("case line resident adjoint", kind, nz, flush=True)
    _adjoint_vs_oracle(_case(kind, nz), 3)
