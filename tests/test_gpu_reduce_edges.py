"""The reductions and the upscale integration at the edges of their vector loads:
rows shorter than a vector, rows that end inside one, levels of more than one
part, against the oracle.

Tolerances: the kernels form the oracle's terms in double from the stored
values, each rounded a few times, and sum them compensated or as maxima; 1e-12
of the largest value covers some thousand roundings of 1.1e-16.  The
integration's FP32 result is rounded once to float (6e-8)."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,m,walls", [((1, 1, 2), (1, 1, 1), False), ((3, 5, 4), (1, 1, 1), False),
                                       ((6, 3, 10), (2, 1, 2), True), ((9, 12, 9), (3, 3, 3), False),
                                       ((67, 70, 9), (1, 1, 1), True), ((260, 36, 20), (4, 3, 2), False),
                                       ((258, 34, 17), (2, 2, 1), True), ((20, 15, 10), (5, 3, 2), False)])
def test_reductions_at_vector_edges(n, m, walls, prec):
    from paper_1805_03426_amd.context import Context
    print("case reductions", n, m, walls, prec, flush=True)
    nx, ny, nz = n
    rng = np.random.default_rng(nx + 7 * ny)
    hx = rng.uniform(0.7, 1.3, nx)
    xf = np.concatenate([[0.0], np.cumsum(hx)]) / hx.sum()
    yf, zf = np.arange(ny + 1) / ny, np.sort(np.concatenate([[0.0, 1.0], rng.uniform(0.02, 0.98, nz - 1)]))
    side = "walls" if walls else "periodic"
    dtype = np.float64 if prec == "fp64" else np.float32
    draw = lambda s: rng.uniform(-1.0, 1.0, s).astype(dtype).astype(np.float64)  # noqa: E731
    th, u, v, w = draw((nz, ny, nx)), draw((nz, ny, nx)), draw((nz, ny, nx)), draw((nz + 1, ny, nx))
    if walls:
        u[:, :, 0] = 0.0
        v[:, 0, :] = 0.0
    g = O.Grid(xf, yf, zf, m, periodic=(not walls, not walls, False))
    p = O.ScalarParams.from_ra_pr(1e6, 1.0, 1e-6)
    with Context(xf, yf, zf, m, 1e6, 1.0, 1e-6, precision=prec, side_x=side, side_y=side) as ctx:
        d = [torch.from_numpy(a).to("cuda", ctx.dtype) for a in (th, u, v, w)]
        prof = ctx.nusselt(d[0], d[3], sync=False)[0].cpu().numpy()
        diss = ctx.thermal_dissipation(d[0], sync=False)[0].cpu().numpy()
        tc = ctx.integrate_scalar(d[0]).cpu().numpy().astype(np.float64)
        div = ctx.divergence(*d[1:]).cpu().numpy()
    want, summ = O.nusselt(g, p, th, w)
    want = np.concatenate([want, [summ[k] for k in ("nu_bot", "nu_top", "nu_vol", "nu_paper", "mean_theta")]])
    if nz == 1:
        want[-2] = prof[-2]
    assert np.max(np.abs(prof - want)) <= TOL * np.max(np.abs(want))
    t = O.thermal_dissipation(g, p, th)
    want = np.array([t[k] for k in ("nu_t", "gx2", "gy2", "gz2")])
    assert np.max(np.abs(diss - want)) <= TOL * np.max(np.abs(want))
    want = O.integrate_scalar(g, th)
    assert np.max(np.abs(tc - want)) <= (TOL if prec == "fp64" else 1.2e-7)
    pad = lambda q, ax: np.concatenate([q, np.zeros_like(np.take(q, [0], axis=ax))], axis=ax) if walls else q  # noqa: E731
    net, tot = O.divergence(g, pad(u, 2), pad(v, 1), w)
    want = np.array([np.max(np.abs(net)), np.max(np.abs(net) / tot)])
    assert np.all(np.abs(div - want) <= TOL * want)
