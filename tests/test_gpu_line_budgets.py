"""GPU parity of the line solver's columns of 9 to 12 chunks, whose kernels are
compiled for 768 or 1024 threads by precision and face order: stretched y, side
walls, explicit z share and fourth-order faces.  Tolerances: those of the step and
adjoint tests."""
import pytest

from tests.test_gpu_face4 import Case4, _adjoint_vs_oracle, _steps
from tests.test_gpu_parity import FP32_TOL, FP64_TOL
from tests.test_gpu_zweight import ZCase

pytestmark = pytest.mark.gpu
KINDS = {"stretched": (2, (False, False), 0.0), "walls": (2, (True, True), 0.0), "explicit z": (2, (False, False), 0.5),
         "fourth order": (4, (False, False), 0.0)}


def _case(kind, nz, prec):
    order, walls, wz = KINDS[kind]
    kw = dict(precision=prec, n_avg=3, dt=1e-3)
    if order == 4:
        return Case4((6, 12, nz), (1, 1, 1), walls, z_explicit=wz, **kw)
    return ZCase((6, 12, nz), (1, 1, 1), walls, wz, **kw)


@pytest.mark.parametrize("nz", [257, 384, 385])
@pytest.mark.parametrize("kind", list(KINDS))
def test_budgets(kind, nz):
    for prec, tol in (("fp64", FP64_TOL), ("fp32", FP32_TOL)):
        print("case line budgets", kind, nz, prec, flush=True)
        _steps(_case(kind, nz, prec), 3, tol)
    _adjoint_vs_oracle(_case(kind, nz, "fp64"), 3)
