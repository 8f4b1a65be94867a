"""The reverse sweep in blocks of several waves (more than 2^16 particles), with
several steps a launch: grid gradients at the box regimes a launch can meet --
boxes that fit, that are cut down, and that are left out, where the steps of a
launch follow one another without a box between them.

Bounds as in the other derivative tests: 1e-9 relative to the largest adjoint
and 1e-10 to the largest grid entry against the oracle's full-tape reverse sweep
(the same FP64 map, other rounding and summation order); the fixed-point
gradient has the same bits at every block size."""
import functools

import numpy as np
import pytest

import oracle
from paper_2607_17836_amd import lpt, synth

pytestmark = pytest.mark.gpu

COUNT = (1 << 16) + 4321   # above the one-wave blocks' line, ragged


def _scale(a):
    return max(1.0, float(np.max(np.abs(a))))


@functools.lru_cache(maxsize=None)
def _case(scheme, n, cells):
    """Fields, particles, cotangents and the oracle's gradients."""
    steps, dt = 19, cells * 2 * np.pi / n   # more steps than a launch takes
    u, v, _ = synth.taylor_green(n)
    (pa, qa), (pb, qb) = synth.spectrum_snapshots(n, 2, 3, dt)
    fields = ((u + 0.2 * pa, v + 0.2 * qa), (u + 0.2 * pb, v + 0.2 * qb))
    x, y = oracle.init_uniform(23, COUNT)
    rng = np.random.default_rng(15)
    a, b = rng.normal(size=COUNT), rng.normal(size=COUNT)
    fl = oracle.grid_flow(*fields[0], *fields[1], scheme=scheme, time_mode=oracle.BRACKET,
                          t_slot=(0.0, steps * dt))
    return steps, dt, fields, x, y, a, b, oracle.adjoint(fl, x, y, a, b, steps, dt)


# n, step in cells at speed 1, re-sort, tile: sorted and dense (boxes fit);
# sorted, sparser and fast (cut down); sparser still, in the larger LDS; unsorted,
# so that every block's box is the whole grid: cut down to a window on 96^2, left
# out on 320^2, with tiles and, so that their barriers fall away too, without
@pytest.mark.parametrize("scheme", ["bilinear", "bspline"])
@pytest.mark.parametrize("n,cells,interval,tile", [(96, 1.0, 5, 0), (320, 6.0, 5, 0),
                                                   (640, 1.0, 5, 0), (96, 1.0, 0, 0),
                                                   (96, 1.0, 0, -1), (320, 6.0, 0, 0),
                                                   (320, 6.0, 0, -1)])
def test_grid_gradient_of_multi_wave_blocks(scheme, n, cells, interval, tile):
    steps, dt, fields, x, y, a, b, (ox, oy, oU) = _case(scheme, n, cells)
    ref = None
    for det in (True, False):
        for block in (128, 256, 512):
            print(f"multi-wave gradient {scheme} n={n} interval={interval} tile={tile} "
                  f"det={det} block={block}", flush=True)
            tr = lpt.Tracker(n, "fp64", sort_interval=interval, block_size=block,
                             tile_records=tile, deterministic_grad=det)
            tr.set_snapshot(0, 0.0, *fields[0])
            tr.set_snapshot(1, steps * dt, *fields[1])
            tr.add_species("tracer", 0.0, scheme, x, y)
            tr.forward_checkpointed(steps, dt, steps - 1)   # and a segment of one step
            gx, gy, gU = tr.adjoint(a, b)
            tr.close()
            assert np.max(np.abs(gx - ox)) < 1e-9 * _scale(ox)
            assert np.max(np.abs(gy - oy)) < 1e-9 * _scale(oy)
            assert np.max(np.abs(gU - oU)) < 1e-10 * _scale(oU)
            if ref is None:
                ref = gx, gy, gU
            np.testing.assert_array_equal(gx, ref[0])
            np.testing.assert_array_equal(gy, ref[1])
            if det:
                np.testing.assert_array_equal(gU, ref[2])
