"""The FP32 velocity gradient on both sides of its rule's lines: rounds of the large
form's workgroups (64 x 8 columns, 16 levels) filled to 4/5 or more, one, two and
three rounds.  Reference and tolerances: those of the gradient's forms."""
import pytest

from tests.test_gpu_grad_forms import test_velocity_gradient_forms as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(64, 405, 127), (60, 411, 128), (64, 512, 128), (63, 505, 129), (64, 504, 207), (64, 505, 208),
                               (64, 1024, 129)])
@pytest.mark.parametrize("count", [3, 8, 10])
def test_rounds(n, count):
    check(n, count)
