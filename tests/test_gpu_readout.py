"""Readout of positions and velocities out of cell order: the two-pass readout
of large reordered species against the one-pass readout of the same state in
its original order (sorting only moves slots, so every value is the same bits)."""
import numpy as np
import pytest

from paper_2607_17836_amd import lpt, synth

pytestmark = pytest.mark.gpu

POS, VEL = 1 << 19, 1 << 20   # the smallest species that take the two passes


def _read(tr, sid, which):
    import torch
    out = [torch.full((tr.counts[sid],), float("nan"), dtype=torch.float64, device="cuda")
           for _ in range(4)]
    tr.get_positions(sid, out=[o if w else None for o, w in zip(out, which)])
    tr.synchronize()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("count", [POS - 1, POS, POS + 77, VEL, VEL + 1])
def test_sorted_readout_equals_unsorted(precision, count):
    n = 48
    u, v, _ = synth.taylor_green(n)
    tr = lpt.Tracker(n, precision)
    tr.set_snapshot(0, 0.0, u, v)
    tr.set_snapshot(1, 1.0, u, v)
    x0, y0 = synth.random_points(count + 131, seed=3)
    # a first species of odd size, so that the second starts at an odd offset
    a = tr.add_species("tracer", 0.0, "bilinear", x0[:131], y0[:131])
    b = tr.add_species("inertial", 0.5, "bilinear", x0[131:], y0[131:])
    tr.step(3, 0.05)
    every = (True, True, True, True)
    before = [_read(tr, s, every) for s in (a, b)]
    vel = tr.get_velocities(b)
    tr.sort()
    assert not np.array_equal(tr.get_order(b), np.arange(count))
    for s, ref in zip((a, b), before):
        for got, want in zip(_read(tr, s, every), ref):
            assert np.array_equal(got, want)
    # outputs left out stay untouched, the others are unchanged
    for which in ((True, False, False, False), (False, True, True, False)):
        for got, want, w in zip(_read(tr, b, which), before[1], which):
            assert np.array_equal(got, want) if w else np.isnan(got).all()
    # host arrays, and the velocities
    for got, want in zip(tr.get_positions(b), before[1]):
        assert np.array_equal(got, want)
    for got, want in zip(tr.get_velocities(b), vel):
        assert np.array_equal(got, want)
    # the scratch of a readout is no state: the next steps are those of a
    # tracker that read nothing
    tr.step(2, 0.05)
    after = _read(tr, b, every)
    tr.close()
    ref = lpt.Tracker(n, precision)
    ref.set_snapshot(0, 0.0, u, v)
    ref.set_snapshot(1, 1.0, u, v)
    ref.add_species("tracer", 0.0, "bilinear", x0[:131], y0[:131])
    ref.add_species("inertial", 0.5, "bilinear", x0[131:], y0[131:])
    ref.step(5, 0.05)
    for got, want in zip(after, _read(ref, b, every)):
        assert np.array_equal(got, want)
    ref.close()
