"""The fused refinement at the edges of its work split: x factors with one lane
per coarse cell (1 to 4) and per dense column (5), tiles narrowed by walls,
ragged tiles and layer ranges, small grids with one layer per workgroup and
larger ones with several, y factors past the product that replaces a division.
Against the oracle at the tolerances of the other refinement tests; nothing
outside the outputs is written."""
import numpy as np
import pytest
import torch

import oracle as O
from tests.test_gpu_parity import FP32_TOL, FP64_TOL, host, rel_max
from tests.test_gpu_walls import WallCase

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,m,walls", [
    ((33, 6, 5), (1, 1, 1), (False, False)), ((65, 11, 4), (1, 2, 2), (True, True)),
    ((33, 7, 4), (2, 2, 2), (True, False)), ((64, 160, 24), (2, 1, 1), (False, False)),
    ((22, 6, 3), (3, 3, 3), (True, True)), ((43, 5, 7), (3, 2, 4), (False, True)),
    ((17, 13, 4), (4, 3, 2), (True, True)), ((15, 7, 3), (4, 4, 4), (False, False)),
    ((13, 6, 3), (5, 2, 2), (False, True)), ((3, 3, 3), (2, 70, 1), (False, False)),
])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_refine_work_split_edges(nc, m, walls, prec):
    print("case refine edges", nc, m, walls, prec, flush=True)
    c = WallCase(nc, m, walls, precision=prec, dt=1e-6)
    U, V, W = c.coarse_velocity()
    want = O.refine_velocity(c.g, U, V, W)
    Ul, Vl = c.to_lib(U, V)
    pad = 64
    with c.ctx() as ctx:
        bufs, outs = [], []
        for shape in (ctx.shape_cell, ctx.shape_cell, ctx.shape_w):
            n = int(np.prod(shape))
            b = torch.full((n + 2 * pad,), 7.25, dtype=c.dtype, device="cuda")
            bufs.append(b)
            outs.append(b[pad:pad + n].view(shape))
        ctx.interpolate_velocity(c.d(Ul), c.d(Vl), c.d(W), out=outs)
        got = [host(t) for t in outs]
        for b in bufs:
            assert bool((b[:pad] == 7.25).all()) and bool((b[-pad:] == 7.25).all())
    gu, gv = c.to_oracle(got[0], got[1])
    for a, b in zip((gu, gv, got[2]), want):
        assert rel_max(a, b) <= (FP64_TOL if prec == "fp64" else FP32_TOL)
