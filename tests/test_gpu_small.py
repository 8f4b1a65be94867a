"""Launches of several steps against launches of one, and the small-population
kernels (no tile, a bicubic stencil split over four lanes) against the tiled ones: a particle's trajectory does not
depend on the population it is part of, so the leading particles of a large
species, which takes the tiled kernels, must have the same bits as the same
particles alone."""
import numpy as np
import pytest

from paper_2607_17836_amd import lpt, synth

pytestmark = pytest.mark.gpu

# one particle more than the largest population the small kernels take
LARGE = (1 << 18) + 1


def _tracker(n, precision, mode, species, **kw):
    u, v, _ = synth.taylor_green(n)
    a, b = synth.spectrum_snapshots(n, 4.0, 9, 0.02)
    dt = 0.02
    tr = lpt.Tracker(n, precision, **kw)
    tr.set_time_mode(mode)
    tr.set_snapshot(0, 0.0, u + 0.3 * a[0], v + 0.3 * a[1])
    tr.set_snapshot(1, dt if mode == "pingpong" else 100 * dt, u + 0.3 * b[0], v + 0.3 * b[1])
    for kind, st, scheme, x, y in species:
        tr.add_species(kind, st, scheme, x, y)
    return tr, dt


def _state(tr, sid, inertial, m):
    out = [a[:m] for a in tr.get_positions(sid)]
    return out + ([a[:m] for a in tr.get_velocities(sid)] if inertial else [])


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("scheme", ["bilinear", "catmull_rom", "bspline"])
@pytest.mark.parametrize("mode,compat,interval", [("pingpong", False, 0), ("bracket", False, 7),
                                                  ("bracket", True, 0)])
def test_small_equals_tiled(precision, scheme, mode, compat, interval):
    n, steps = 40, 21   # more steps than one launch takes
    x, y = synth.random_points(LARGE, seed=5)
    for count in (1, 63, 64, 65, 1000):
        got = {}
        for size in (count, LARGE):
            species = [("tracer", 0.0, scheme, x[:size], y[:size]),
                       ("inertial", 0.3, scheme, x[:count], y[:count])]
            tr, dt = _tracker(n, precision, mode, species, compat_edge=compat,
                              sort_interval=interval)
            tr.step(steps, dt, stats_every=5)
            got[size] = (_state(tr, 0, False, count), _state(tr, 1, True, count),
                         tr.get_stats(1), tr.get_time())
            tr.close()
        small, large = got[count], got[LARGE]
        for s in (0, 1):
            for p, q in zip(small[s], large[s]):
                assert np.array_equal(p, q), (count, s)
        assert small[3] == large[3]
        assert len(small[2]) == steps // 5
        # the same slots summed in the same order; a re-sort orders equal keys
        # by slot, which does not depend on the other species
        for f in small[2].dtype.names:
            assert np.array_equal(small[2][f], large[2][f]), (count, f)


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("scheme", ["bilinear", "catmull_rom", "mixed"])
@pytest.mark.parametrize("tuning", [dict(), dict(block_size=512, rows=2), dict(tile_records=-1),
                                    dict(tile_records=64, block_size=128), dict(fused=0),
                                    dict(persistent=1, max_workgroups=64)])
def test_runs_equal_single_steps(precision, scheme, tuning):
    """The tiled kernels: 21 steps in one call (runs of up to 16, cut by records
    and re-sorts) against 21 calls of one step."""
    n, steps, count = 40, 21, LARGE + 50
    x, y = synth.random_points(count + 3000, seed=6)
    first = "bilinear" if scheme == "mixed" else scheme
    second = "bspline" if scheme == "mixed" else scheme
    species = [("tracer", 0.0, first, x[:count], y[:count])]
    if scheme != "bilinear":   # one species alone takes its own kernels
        species.append(("inertial", 0.3, second, x[count:], y[count:]))
    got = []
    for single in (False, True):
        tr, dt = _tracker(n, precision, "bracket", species, sort_interval=18)
        tr.set_tuning(**tuning)
        if single:
            for _ in range(steps):
                tr.step(1, dt, stats_every=20)
        else:
            tr.step(steps, dt, stats_every=20)
        out = [_state(tr, s, s == 1, count) for s in range(len(species))]
        got.append((sum(out, []), [tr.get_stats(s) for s in range(len(species))],
                    [tr.get_order(s) for s in range(len(species))], tr.get_time()))
        tr.close()
    for p, q in zip(got[0][0], got[1][0]):
        assert np.array_equal(p, q)
    for k in (1, 2):
        for p, q in zip(got[0][k], got[1][k]):
            assert np.array_equal(p, q)
    assert got[0][3] == got[1][3]


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("nspecies", [1, 2, 5])
def test_small_statistics_and_launch_lengths(precision, nspecies):
    """Records of small species (merged by one launch) against the positions,
    and runs of steps against single steps."""
    n, count = 32, 777
    x, y = synth.random_points(count * nspecies, seed=8)
    species = [("tracer", 0.0, ("bilinear", "bspline")[s % 2], x[s * count:(s + 1) * count],
                y[s * count:(s + 1) * count]) for s in range(nspecies)]
    tr, dt = _tracker(n, precision, "pingpong", species, sort_interval=8)
    one, _ = _tracker(n, precision, "pingpong", species, sort_interval=8)
    tr.step(40, dt, stats_every=20)
    for _ in range(40):
        one.step(1, dt, stats_every=20)
    for s in range(nspecies):
        pos = tr.get_positions(s)
        for p, q in zip(pos, one.get_positions(s)):
            assert np.array_equal(p, q)
        rec = tr.get_stats(s)
        assert len(rec) == 2 and np.array_equal(rec, one.get_stats(s))
        xs, ys = species[s][3:]
        r2 = (pos[2] - xs) ** 2 + (pos[3] - ys) ** 2
        # sums of `count` binary64 terms: count * 2^-53 relative, doubled for
        # the differences of positions (xu - x0 rounds at 2^-53 of L)
        assert abs(rec["msd"][1] - r2.mean()) <= 1e-11 * r2.mean()
        sem = np.sqrt(r2.var(ddof=1) / count)
        assert abs(rec["sem"][1] - sem) <= 1e-11 * sem
    tr.close()
    one.close()


@pytest.mark.parametrize("scheme", ["bilinear", "bspline"])
def test_small_checkpointed_run(scheme):
    """Segment lengths that do not divide the launches' step count."""
    n, steps = 32, 37
    x, y = synth.random_points(500, seed=4)
    ref = None
    for every in (37, 5, 18):
        tr, dt = _tracker(n, "fp64", "bracket", [("tracer", 0.0, scheme, x, y)])
        tr.forward_checkpointed(steps, dt, every)
        out = list(tr.get_positions(0)) + [tr.jacobian()]
        tr.close()
        if ref is None:
            ref = out
        for p, q in zip(out, ref):
            assert np.array_equal(p, q)
