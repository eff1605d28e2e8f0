"""GPU parity of the streaming step (one walk per step, truncated look-ahead):
every step type and the reverse step at the edges of its tiles, segments,
copies and look-aheads.

The look-ahead depends on r = tau kappa / h_z^2: with uniform z spacing the
factor per level is x = (1 + 2 r - sqrt(1 + 4 r)) / (2 r), so r = 0.05, 0.3, 0.9
and 2 need about 13, 24, 41 and 57 levels (one per compiled look-ahead) and
r = 5 more than any of them (the line solver, or column sweeps on tall columns).

Tolerances.  FP64: a result is a combination with weights of at most 1 of
right-hand sides of about 40 terms of size at most 4, each rounded once or
twice: 100 eps x 4 = 9e-14, taken as 1e-13.  FP32: the streaming step forms the
same float right-hand sides as the line solver and the column sweeps, and
eliminates in double; a stored float differs only where the doubles, 1e-14
apart at most, straddle a rounding boundary (1e-14 / 6e-8 per value): fewer
than one value in 10^4 differs after a step, and by one float spacing.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

RA, PR, N_AVG = 1e6, 1.0, 4
KAPPA = (RA * PR) ** -0.5
KDT = 1e-5                       # kappa dt


def _faces(nx, ny, nz, r):
    hz = np.sqrt(2.0 * KDT / r)
    # x and y widths of 1/32 (the explicit diffusion number 16 kappa dt 32^2 is 0.16)
    return np.arange(nx + 1) / 32, np.arange(ny + 1) / 32, np.arange(nz + 1) * hz


def _case(nx, ny, nz, r, seed=5):
    xf, yf, zf = _faces(nx, ny, nz, r)
    rng = np.random.default_rng(seed)
    dt = KDT / KAPPA
    # face velocities with tau |u| / h of about 0.3
    u, v = (rng.uniform(-0.15, 0.15, (nz, ny, nx)) * h / dt for h in (xf[1], yf[1]))
    w = rng.uniform(-0.15, 0.15, (nz + 1, ny, nx)) * zf[1] / dt
    w[0] = w[-1] = 0.0
    th = [rng.uniform(-1.0, 1.0, (nz, ny, nx)) for _ in range(3)]
    return (xf, yf, zf), dt, (u, v, w), th


def _ctx(faces, dt, prec, method="auto"):
    from paper_1805_03426_amd.context import Context
    return Context(*faces, (1, 1, 1), RA, PR, dt, n_avg=N_AVG, precision=prec, step_method=method)


def _dev(ctx, arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).to("cuda", ctx.dtype) for a in arrays]


@pytest.mark.parametrize("nx,ny,nz,r", [
    (2, 1, 1, 0.05), (2, 2, 3, 0.05), (64, 4, 8, 0.05), (66, 5, 7, 0.05), (62, 3, 9, 0.3), (130, 9, 40, 0.05),
    (258, 13, 33, 0.05), (128, 64, 100, 0.3), (34, 18, 130, 0.9), (192, 8, 90, 0.9), (66, 6, 150, 2.0),
    (40, 10, 120, 5.0), (62, 7, 700, 0.3), (63, 7, 700, 0.9), (5, 3, 650, 2.0), (1, 1, 700, 0.05), (30, 8, 660, 5.0),
])
def test_stream_steps_fp64(nx, ny, nz, r):
    """Start-up, leapfrog (walking up and down) and averaging steps against the
    oracle; the tall columns also with odd N_x (copies of 4 bytes)."""
    print("case stream fp64", nx, ny, nz, r, flush=True)
    faces, dt, uvw, th = _case(nx, ny, nz, r)
    g = O.Grid(*faces, (1, 1, 1))
    p = O.ScalarParams.from_ra_pr(RA, PR, dt, n_avg=N_AVG)
    with _ctx(faces, dt, "fp64") as ctx:
        duvw, dth = _dev(ctx, uvw), _dev(ctx, th)
        for n in (0, 1, 2, 3):
            out = ctx.scalar_step(n, dth[0], dth[1], ctx.empty(ctx.shape_cell), *duvw)
            want = O.scalar_step(g, p, n, th[0], th[1], *uvw)
            err = np.max(np.abs(out.cpu().numpy() - want))
            assert err <= 1e-13, (n, err)


@pytest.mark.parametrize("nx,ny,nz,r", [
    (2, 2, 3, 0.05), (66, 5, 7, 0.05), (130, 9, 40, 0.3), (258, 13, 33, 0.05), (34, 18, 130, 0.9), (66, 6, 150, 2.0),
    (63, 7, 700, 0.3), (30, 8, 660, 2.0),
])
def test_stream_reverse_steps_fp64(nx, ny, nz, r):
    """Reverse steps (n = 1: down, n = 2: up; n = 3 averages; without a step
    n + 1 and with one) against the oracle's vector-Jacobian product: with
    lam^n = mu^{n+1}'s share through its lag + C_u^T mu^n + a_c mu^n, the result
    is the transposed solve of step n - 1."""
    print("case stream reverse fp64", nx, ny, nz, r, flush=True)
    faces, dt, uvw, th = _case(nx, ny, nz, r, seed=6)
    g = O.Grid(*faces, (1, 1, 1))
    p = O.ScalarParams.from_ra_pr(RA, PR, dt, n_avg=N_AVG)

    def vjp(n, mu):
        """(share of theta^{n-1}, share of theta^n) of step n from mu^n itself."""
        tau, _, _, _ = O.step_kind(n, N_AVG, dt)
        sub, diag, sup, _ = O.z_matrix(g, tau * p.kappa, p)
        # lam = Z^T mu, so that the product's own transposed solve returns mu
        lam = diag[:, None, None] * mu
        lam[:-1] += sub[1:, None, None] * mu[1:]
        lam[1:] += sup[:-1, None, None] * mu[:-1]
        return O.step_vjp(g, p, n, th[2], *uvw, lam)[:2]

    with _ctx(faces, dt, "fp64") as ctx:
        duvw, dth = _dev(ctx, uvw), _dev(ctx, th)
        for n, has_next in ((1, True), (2, True), (3, False), (2, False)):
            out = ctx.scalar_step_backward(n, dth[0] if has_next else None, dth[1], None,
                                           ctx.empty(ctx.shape_cell), *duvw)
            lam = vjp(n, th[1])[1]
            if has_next:
                lam = lam + vjp(n + 1, th[0])[0]
            tau, _, _, _ = O.step_kind(n - 1, N_AVG, dt)
            sub, diag, sup, _ = O.z_matrix(g, tau * p.kappa, p)
            want = O.thomas(np.append(0.0, sup[:-1]), diag, np.append(sub[1:], 0.0), lam)
            err = np.max(np.abs(out.cpu().numpy() - want))
            assert err <= 1e-13, (n, has_next, err)


@pytest.mark.parametrize("nx,ny,nz,r,method", [
    (256, 140, 128, 0.05, "line"), (201, 160, 150, 0.3, "line"), (132, 9, 700, 0.3, "sweep"), (61, 7, 650, 0.9, "sweep"),
])
def test_stream_fp32_matches_line_solver_and_sweeps(nx, ny, nz, r, method):
    """FP32: one float spacing in at most one value in 10^4 after one step, in a
    sequence (the sweeps' walk directions) and in a single step."""
    print("case stream fp32", nx, ny, nz, r, method, flush=True)
    faces, dt, uvw, th = _case(nx, ny, nz, r)
    got = {}
    for m in ("auto", method):
        with _ctx(faces, dt, "fp32", m) as ctx:
            duvw, dth = _dev(ctx, uvw), _dev(ctx, th)
            one = ctx.scalar_step(2, dth[0], dth[1], ctx.empty(ctx.shape_cell), *duvw)
            seq = ctx.scalar_steps(0, None, dth[1], [ctx.empty(ctx.shape_cell) for _ in range(2)], *duvw)
            # the second step alone, from the same first level
            got[m] = [one, seq[0], seq[1]]
    for q, (a, b) in enumerate(zip(got["auto"], got[method])):
        differ = float((a != b).float().mean())
        # the sequence's second step also sees the first one's differences (7 cells each)
        assert differ <= (8e-4 if q == 2 else 1e-4), (q, differ)
        assert float((a - b).abs().max()) <= 2.5e-7, q
