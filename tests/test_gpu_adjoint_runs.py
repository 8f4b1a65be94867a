"""The reverse sweep's launches of several steps and its gradient boxes, at the
sizes where they change: segments longer than one launch and not a multiple of
it, one-step segments, blocks of one wave, boxes that need more LDS than the
default, are cut down or left out, and grids that a box wraps around.

Against the oracle's full-tape reverse sweep, within the bounds of the other
derivative tests: 1e-9 relative to the largest adjoint, 1e-10 to the largest
grid entry (both sides differentiate the same FP64 map and differ in rounding
and summation order)."""
import numpy as np
import pytest

import oracle
from paper_2607_17836_amd import lpt, synth

pytestmark = pytest.mark.gpu


def _scale(a):
    return max(1.0, float(np.max(np.abs(a))))


def _run(n, scheme, x, y, fields, dt, steps, every, a, b, **kw):
    (ua, va), (ub, vb) = fields
    tr = lpt.Tracker(n, "fp64", **kw)
    tr.set_snapshot(0, 0.0, ua, va)
    tr.set_snapshot(1, steps * dt, ub, vb)
    tr.add_species("tracer", 0.0, scheme, x, y)
    tr.forward_checkpointed(steps, dt, every)
    out = tr.adjoint(a, b)
    gx, gy, none = tr.adjoint(a, b, want_grid=False)
    assert none is None
    # without the grid gradient the same adjoints
    assert np.array_equal(gx, out[0]) and np.array_equal(gy, out[1])
    F = tr.jacobian()
    tr.close()
    return out + (F,)


# n, particles, step in cells at speed 1, re-sort: (8) a box wider than the grid;
# (64, 300) scattered blocks of one wave, whose boxes are left out; (64, 3600)
# sorted blocks of one wave; (200, 10000) sorted and sparse, boxes of the larger
# LDS; (200, 2500) sparser than any LDS holds, cut down or left out
@pytest.mark.parametrize("scheme", ["bilinear", "bspline"])
@pytest.mark.parametrize("n,count,cells,interval", [(8, 200, 0.4, 0), (64, 300, 1.5, 0),
                                                    (64, 3600, 2.5, 5), (200, 10000, 1.0, 5),
                                                    (200, 2500, 6.0, 5)])
@pytest.mark.parametrize("det", [False, True])
def test_gradient_boxes_match_oracle(scheme, n, count, cells, interval, det):
    steps = 19   # more than a launch takes
    dt = cells * 2 * np.pi / n
    u, v, _ = synth.taylor_green(n)
    (pa, qa), (pb, qb) = synth.spectrum_snapshots(n, 2, 3, dt)
    fields = ((u + 0.2 * pa, v + 0.2 * qa), (u + 0.2 * pb, v + 0.2 * qb))
    x, y = oracle.init_uniform(17, count)
    rng = np.random.default_rng(5)
    a, b = rng.normal(size=count), rng.normal(size=count)
    fl = oracle.grid_flow(*fields[0], *fields[1], scheme=scheme, time_mode=oracle.BRACKET,
                          t_slot=(0.0, steps * dt))
    ox, oy, oU = oracle.adjoint(fl, x, y, a, b, steps, dt)
    ref = None
    for every in (1, 6, 18, steps):
        gx, gy, gU, F = _run(n, scheme, x, y, fields, dt, steps, every, a, b,
                             sort_interval=interval, deterministic_grad=det)
        assert np.max(np.abs(gx - ox)) < 1e-9 * _scale(ox)
        assert np.max(np.abs(gy - oy)) < 1e-9 * _scale(oy)
        assert np.max(np.abs(gU - oU)) < 1e-10 * _scale(oU)
        if ref is None:
            ref = gx, gy, F
        for p, q in zip((gx, gy, F), ref):   # independent of the segments
            assert np.array_equal(p, q)


@pytest.mark.parametrize("scheme", ["bilinear", "catmull_rom"])
def test_sweep_block_sizes_agree(scheme):
    """Populations on both sides of the one-wave blocks' line (2^16): the same
    particles have the same adjoints and Jacobians."""
    n, steps, few, many = 96, 8, 5000, (1 << 16) + 4000
    dt = 0.05
    u, v, _ = synth.taylor_green(n)
    x, y = oracle.init_uniform(29, many)
    rng = np.random.default_rng(6)
    a, b = rng.normal(size=many), rng.normal(size=many)
    small = _run(n, scheme, x[:few], y[:few], ((u, v), (u, v)), dt, steps, 3, a[:few], b[:few])
    large = _run(n, scheme, x, y, ((u, v), (u, v)), dt, steps, 3, a, b)
    for k in (0, 1, 3):
        assert np.array_equal(small[k], large[k][:few])
