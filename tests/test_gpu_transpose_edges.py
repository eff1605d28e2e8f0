"""The transposed refinement where the last range of coarse layers (along z) or
of coarse rows (along a walled y) that one thread walks holds a single one.
FP64 against the oracle; the tolerance of the other refinement tests."""
import pytest

import oracle as O
from tests.test_gpu_parity import FP64_TOL, host, rel_max
from tests.test_gpu_walls import WallCase

pytestmark = pytest.mark.gpu


def transpose_vs_oracle(nc, m, walls):
    c = WallCase(nc, m, walls, dt=1e-7)
    u, v, w = c.dense_velocity()
    want = O.refine_velocity_transpose(c.g, u, v, w)
    ul, vl = c.to_lib(u, v)
    with c.ctx() as ctx:
        got = [host(t) for t in ctx.interpolate_velocity_backward(c.d(ul), c.d(vl), c.d(w))]
    gU, gV = want[0], want[1]
    # the wall faces carry no velocity: the library keeps no gradient there
    gU = gU[:, :, :-1].copy() if walls[0] else gU
    gV = gV[:, :-1].copy() if walls[1] else gV
    if walls[0]:
        gU[:, :, 0] = 0.0
    if walls[1]:
        gV[:, 0] = 0.0
    for a, b in zip(got, (gU, gV, want[2])):
        assert rel_max(a, b) <= FP64_TOL


@pytest.mark.parametrize("nc,m,walls", [
    ((3, 2, 1), (1, 1, 1), (False, False)), ((3, 3, 1), (2, 2, 1), (True, True)),
    ((3, 2, 241), (1, 1, 1), (False, False)), ((3, 4, 257), (2, 1, 2), (False, True)),
    ((3, 993, 3), (2, 2, 2), (True, True)), ((3, 993, 2), (1, 1, 1), (False, True)),
])
def test_transposed_refinement_single_last_layer_or_row(nc, m, walls):
    print("case transpose edges", nc, m, walls, flush=True)
    transpose_vs_oracle(nc, m, walls)
