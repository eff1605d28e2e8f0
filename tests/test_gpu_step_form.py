"""The form in which a context runs its steps, as the library reports it: forced
methods, columns beyond the line solver, the variants' forward step alone, and
grids that a listed form is the fastest on by a wide margin."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
CALLS = ("scalar_step", "scalar_steps", "scalar_step_backward", "scalar_steps_backward")


def _ctx(n, r=0.05, **kw):
    from paper_1805_03426_amd.context import Context
    # widths of 1/32 in x and y, kappa dt = 1e-5, tau kappa / h_z^2 = r at tau = 2 dt
    faces = [np.arange(n[0] + 1) / 32, np.arange(n[1] + 1) / 32, np.arange(n[2] + 1) * np.sqrt(2e-5 / r)]
    return Context(*faces, (1, 1, 1), 1e6, 1.0, 1e-2, **kw)


def _forms(*args, **kw):
    with _ctx(*args, **kw) as ctx:
        return tuple(ctx.step_form(c) for c in CALLS)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_step_forms(prec):
    print("case step forms", prec, flush=True)
    line, sweep, stream = ("line",) * 4, ("sweep",) * 4, ("stream",) * 4
    assert _forms((64, 64, 64), precision=prec) == line
    assert _forms((256, 256, 256), precision=prec) == stream
    assert _forms((256, 256, 256), precision=prec, step_method="line") == line
    assert _forms((256, 256, 256), precision=prec, step_method="sweep") == ("sweep", "sweep", "line", "sweep")
    assert _forms((32, 8, 700), precision=prec) == stream
    assert _forms((32, 8, 700), r=5.0, precision=prec) == sweep          # look-ahead past 60 levels
    assert _forms((256, 256, 256), precision=prec, side_x="walls") == ("stream", "stream", "line", "line")
    assert _forms((64, 64, 64), precision=prec, face_order=4) == line


def test_unknown_call_is_refused():
    from ctypes import byref, c_int32
    from paper_1805_03426_amd import _lib
    out = c_int32()
    with _ctx((32, 8, 16)) as ctx:
        for call in (-1, 4):
            assert _lib.lib().mr_get_step_form(ctx._ctx, call, byref(out)) == _lib.MR_EINVAL


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_long_look_ahead_takes_the_line_solver(prec):
    """One round of 256 levels: segments of short look-aheads stream faster, of long
    ones (58 levels at r = 2) slower than the line solver."""
    print("case step forms look-ahead", prec, flush=True)
    assert _forms((64, 64, 256), r=0.05, precision=prec) == ("stream",) * 4
    assert _forms((64, 64, 256), r=2.0, precision=prec) == ("line",) * 4
    assert _forms((64, 64, 700), r=2.0, precision=prec) == ("stream",) * 4   # beyond the line solver
