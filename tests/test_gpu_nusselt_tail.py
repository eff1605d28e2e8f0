"""The Nusselt profile's last kernel with one to four partials a level (one lane a
face below four, four lanes from there) and one to several faces a thread, against
the oracle.  Tolerance as for the other reductions: 1e-12 of the largest value
covers some thousand roundings."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 8), (64, 64), (80, 80), (110, 110), (130, 126)])
@pytest.mark.parametrize("nz", [2, 64, 256, 257, 1024])
def test_tail(nx, ny, nz):
    from paper_1805_03426_amd.context import Context
    print("case nusselt tail", nx, ny, nz, flush=True)
    rng = np.random.default_rng(nz + nx)
    xf, yf = np.arange(nx + 1) / nx, np.arange(ny + 1) / ny
    zf = np.sort(np.concatenate([[0.0, 1.0], (np.arange(nz - 1) + rng.uniform(0.75, 1.25, nz - 1)) / nz]))
    th, w = rng.uniform(-1.0, 1.0, (nz, ny, nx)), rng.uniform(-1.0, 1.0, (nz + 1, ny, nx))
    g, p = O.Grid(xf, yf, zf, (1, 1, 1)), O.ScalarParams.from_ra_pr(1e6, 1.0, 1e-7)
    with Context(xf, yf, zf, (1, 1, 1), 1e6, 1.0, 1e-7) as ctx:
        prof = ctx.nusselt(torch.from_numpy(th).cuda(), torch.from_numpy(w).cuda(), sync=False)[0].cpu().numpy()
    want, summ = O.nusselt(g, p, th, w)
    want = np.concatenate([want, [summ[k] for k in ("nu_bot", "nu_top", "nu_vol", "nu_paper", "mean_theta")]])
    assert np.max(np.abs(prof - want)) <= 1e-12 * np.max(np.abs(want))
