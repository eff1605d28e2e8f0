"""Reverse step 0 (the derivative with respect to theta^0) as a streaming step:
FP64 against the oracle's vector-Jacobian product of the start-up step plus step
1's share through its lag, at the edges of tiles, segments, copies and
look-aheads; FP32 against the line solver's.  Tolerances: FP64 1e-13 as the other
streaming tests; FP32 sums of about 40 terms of size at most 4 in another order,
40 eps x 4 = 2e-5."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_stream import N_AVG, PR, RA, _case, _ctx, _dev

pytestmark = pytest.mark.gpu


def _vjp(g, p, n, mu, th, uvw, dt):
    tau, _, _, _ = O.step_kind(n, N_AVG, dt)
    sub, diag, sup, _ = O.z_matrix(g, tau * p.kappa, p)
    lam = diag[:, None, None] * mu
    lam[:-1] += sub[1:, None, None] * mu[1:]
    lam[1:] += sup[:-1, None, None] * mu[:-1]
    return O.step_vjp(g, p, n, th, *uvw, lam)[:2]


@pytest.mark.parametrize("nx,ny,nz,r", [
    (66, 5, 130, 0.05), (34, 18, 130, 0.9), (66, 6, 150, 2.0), (63, 7, 700, 0.3), (258, 130, 3, 0.05),
    (2, 2, 129, 0.3),
])
def test_stream_reverse_step_zero(nx, ny, nz, r):
    print("case stream reverse 0", nx, ny, nz, r, flush=True)
    faces, dt, uvw, th = _case(nx, ny, nz, r, seed=8)
    g = O.Grid(*faces, (1, 1, 1))
    p = O.ScalarParams.from_ra_pr(RA, PR, dt, n_avg=N_AVG)
    with _ctx(faces, dt, "fp64") as ctx:
        duvw, dth = _dev(ctx, uvw), _dev(ctx, th)
        for has_next in (True, False):
            out = ctx.scalar_step_backward(0, dth[0] if has_next else None, dth[1], None,
                                           ctx.empty(ctx.shape_cell), *duvw)
            a, b = _vjp(g, p, 0, th[1], th[2], uvw, dt)
            want = b if a is None else a + b
            if has_next:
                want = want + _vjp(g, p, 1, th[0], th[2], uvw, dt)[0]
            err = np.max(np.abs(out.cpu().numpy() - want))
            assert err <= 1e-13, (has_next, err)


def test_stream_reverse_step_zero_fp32():
    print("case stream reverse 0 fp32", flush=True)
    faces, dt, uvw, th = _case(180, 170, 150, 0.3, seed=9)
    got = []
    for m in ("auto", "line"):
        with _ctx(faces, dt, "fp32", m) as ctx:
            duvw, dth = _dev(ctx, uvw), _dev(ctx, th)
            got.append(ctx.scalar_step_backward(0, dth[0], dth[1], None, ctx.empty(ctx.shape_cell), *duvw))
    assert float((got[0] - got[1]).abs().max()) <= 2e-5
