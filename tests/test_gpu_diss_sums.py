"""The dissipation sums take every column's share into their compensated sums by
itself: shares too small to change their neighbour's in a plain double add up.

All widths and weights are powers of two and every difference and square is
exact in double (24-bit differences), so the mean square of the y differences
over columns of 1, t, t, t with t^2 just below 2^-53 is (1 + 3 t^2) N_y^2 / 4
exactly, and the kernel may round it once: 2^-53."""
from fractions import Fraction

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(256, 4, 4), (512, 8, 16), (128, 4, 8)])
def test_small_columns_are_not_lost(nx, ny, nz):
    from paper_1805_03426_amd.context import Context
    print("case dissipation sums", nx, ny, nz, flush=True)
    t = np.float32(0.98 * 2.0 ** -26.5)
    amp = np.where(np.arange(nx) % 4 == 0, np.float32(0.5), t / np.float32(2))
    th = np.where(np.arange(ny) % 2 == 0, 1, -1)[None, :, None] * np.broadcast_to(amp, (nz, ny, nx))
    faces = [np.arange(n + 1) / n for n in (nx, ny, nz)]
    with Context(*faces, (1, 1, 1), 2.0 ** 20, 1.0, 1e-6, precision="fp32", bc_bot="adiabatic",
                 bc_top="adiabatic") as ctx:
        gy = float(ctx.thermal_dissipation(torch.from_numpy(th.astype(np.float32)).cuda(), sync=False)[0][2])
    exact = (1 + 3 * Fraction(float(t)) ** 2) * ny * ny / 4
    assert abs(Fraction(gy) / exact - 1) <= Fraction(2) ** -53
