"""Sequences on flat grids whose sweep tiles keep the GPU full run as column sweeps,
single steps stream: the same levels from both (sums of about 40 terms of size at most
4 in two orders, FP64 1e-13; FP32 one float spacing of the elimination values: 2.5e-7
a step), and a sequence whose first call is captured streams and allocates nothing."""
import numpy as np
import pytest
import torch

from tests.test_gpu_stream import _case, _ctx, _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,nz", [("fp64", 1), ("fp64", 3), ("fp64", 4), ("fp32", 3), ("fp32", 4), ("fp32", 5)])
def test_sequence_equals_single_steps(prec, nz):
    print("case flat", prec, nz, flush=True)
    n = 512 if prec == "fp64" else 1024   # (FP32 streams from 2.5e6 cells)
    faces, dt, uvw, th = _case(n, n, nz, 0.3)
    flat = nz <= (3 if prec == "fp64" else 4)
    tol = 1e-13 if prec == "fp64" else 1e-6
    with _ctx(faces, dt, prec) as ctx:
        assert ctx.step_form("scalar_step") == "stream"
        for call in ("scalar_steps", "scalar_steps_backward"):
            assert ctx.step_form(call) == ("sweep" if flat else "stream")
        duvw, dth = _dev(ctx, uvw), _dev(ctx, th)

        def new():
            return ctx.empty(ctx.shape_cell)
        # a captured sequence first: nothing is allocated yet
        seq = [new() for _ in range(3)]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.scalar_steps(1, dth[0], dth[1], seq, *duvw)
        one = [dth[0], dth[1]]
        for n in range(1, 4):
            one.append(ctx.scalar_step(n, one[-2], one[-1], new(), *duvw))
        eager = ctx.scalar_steps(1, dth[0], dth[1], [new() for _ in range(3)], *duvw)
        for _ in range(2):
            for t in seq:
                t.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for a, b, c in zip(seq, eager, one[2:]):
                assert float((a - c).abs().max()) <= tol and float((b - c).abs().max()) <= tol
        back = [dth[0], dth[1]]
        for n in range(3, 0, -1):
            back.append(ctx.scalar_step_backward(n, back[-2], back[-1], None, new(), *duvw))
        got = ctx.scalar_steps_backward(3, dth[0], dth[1], [new() for _ in range(3)], *duvw)
        for a, b in zip(got, back[2:]):
            assert float((a - b).abs().max()) <= tol
