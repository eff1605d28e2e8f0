"""The FP32 dissipation with four cells a lane (large grids of whole wide tiles) and
with one: every column's share by itself, at the exactness of the smaller grids, and
ragged rows against 64-bit sums in torch.  Tolerance: terms of relative error at most
9 eps and 1/h of a few eps, compensated, against torch's tree sums of 2.5e7 doubles (a
relative error of at most 25 eps): some 1e-14, taken as 1e-13."""
import numpy as np
import pytest
import torch

from tests.test_gpu_diss_sums import test_small_columns_are_not_lost as check

pytestmark = pytest.mark.gpu


def test_small_columns_on_wide_tiles():
    check(512, 512, 128)


@pytest.mark.parametrize("n", [(450, 300, 200), (225, 600, 190), (511, 400, 130), (640, 400, 100)])
def test_ragged_rows(n):
    from paper_1805_03426_amd.context import Context
    print("case dissipation wide", n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n[0])
    faces = [np.arange(k + 1) / k for k in n]
    with Context(*faces, (1, 1, 1), 1e6, 1.0, 1e-8, precision="fp32", bc_bot="adiabatic", bc_top="adiabatic") as ctx:
        th = torch.rand(ctx.shape_cell, dtype=torch.float32, device="cuda", generator=gen)
        got = ctx.thermal_dissipation(th, sync=False)[0].cpu().numpy()
    t = th.double()
    want = [float(((t - t.roll(1, 2)) ** 2).mean()) * n[0] ** 2, float(((t - t.roll(1, 1)) ** 2).mean()) * n[1] ** 2,
            float(((t[1:] - t[:-1]) ** 2).sum()) / t.numel() * n[2] ** 2]
    for a, b in zip(got[1:], want):
        assert abs(a / b - 1) <= 1e-13
