"""The velocity gradient's forms (segments of 4 and 8 levels, loads ahead or not,
the level below carried or not), which depend on the precision, the number of
steps and the grid: small and large grids around the edges of tiles, segments and
runs, against torch in float64.  Sums of up to 10 terms of size at most 1 x 2: 32
eps x 10 rounding units, 1e-13 (FP64) and 1e-4 (FP32) of the largest gradient."""
import numpy as np
import pytest
import torch

from paper_1805_03426_amd import inputs

pytestmark = pytest.mark.gpu


def _want(ctx, th, mu, taus, hx, hy, hz):
    gu = gv = gw = 0.0
    for t, m, tau in zip(th, mu, taus):
        t, m = t.double(), m.double()
        for axis, h in ((2, hx), (1, hy)):
            q = m / h
            g = tau * 0.5 * (t + t.roll(1, axis)) * (q - q.roll(1, axis))
            if axis == 2:
                gu = gu + g
            else:
                gv = gv + g
        q = m / hz[:, None, None]
        g = torch.zeros(t.shape[0] + 1, *t.shape[1:], dtype=torch.float64, device=t.device)
        g[1:-1] = tau * 0.5 * (t[1:] + t[:-1]) * (q[1:] - q[:-1])
        gw = gw + g
    return gu, gv, gw


@pytest.mark.parametrize("n", [(1, 1, 1), (63, 9, 5), (65, 8, 4), (130, 17, 33), (128, 96, 40), (384, 250, 70),
                               (515, 264, 17)])
@pytest.mark.parametrize("count", [1, 4, 5, 8, 9, 16])
def test_velocity_gradient_forms(n, count):
    from paper_1805_03426_amd.context import Context
    xf, yf, zf = inputs.uniform_faces(n[0]), inputs.uniform_faces(n[1]), inputs.tanh_faces(n[2], 1.2 if n[2] > 1 else 0.0)
    dt = 1e-6
    for prec, tol in (("fp64", 1e-13), ("fp32", 1e-4)):
        print("case grad forms", n, count, prec, flush=True)
        with Context(xf, yf, zf, (1, 1, 1), 1e6, 1.0, dt, n_avg=3, precision=prec) as ctx:
            gen = torch.Generator(device="cuda").manual_seed(count)
            f = [torch.rand(ctx.shape_cell, dtype=torch.float64, device="cuda", generator=gen).to(ctx.dtype)
                 for _ in range(2 * count)]
            steps = list(range(count))
            taus = [dt if q == 0 else (1.5 * dt if (q + 1) % 3 == 0 else 2.0 * dt) for q in steps]
            g = [torch.full(s, 0.25 * dt, dtype=ctx.dtype, device="cuda") for s in
                 (ctx.shape_cell, ctx.shape_cell, ctx.shape_w)]
            ctx.velocity_grad(steps, f[:count], f[count:], *g)
            hz = torch.from_numpy(np.diff(zf)).cuda()
            want = _want(ctx, f[:count], f[count:], taus, 1.0 / n[0], 1.0 / n[1], hz)
            for a, b in zip(g, want):
                b = b + 0.25 * dt
                assert float((a.double() - b).abs().max()) <= tol * float(b.abs().max())
