"""The tiled step kernels at populations that take the small-population kernels
by default: an explicit tile capacity selects the tiled ones, which are held
against the oracle where particles leave the tile and where the bicubic schemes
fall back to bilinear, and against each other over block sizes and graph
replays."""
import numpy as np
import pytest

import oracle
from paper_2607_17836_amd import lpt, synth

pytestmark = pytest.mark.gpu

L = 2 * np.pi


def pdist(a, b):
    d = np.abs(np.asarray(a) - np.asarray(b)) % L
    return np.minimum(d, L - d)


@pytest.mark.parametrize("scheme", ["bilinear", "catmull_rom", "bspline"])
def test_escapees_of_a_tile_match_oracle(scheme):
    """FP64 inertial particles launched far faster than the flow (up to 30 cells a
    step) leave the tile during their stages; both sides run the same FP64 steps,
    so they differ by rounding alone: 1e-10 after ten steps (1e-8 for velocities
    of order 100 / St)."""
    print(f"tile escapees {scheme}", flush=True)
    n, dt, count = 128, 0.002, 6000
    (ua, va), (ub, vb) = synth.spectrum_snapshots(n, 6, 9, dt)
    x0, y0 = oracle.init_uniform(77, count)
    rng = np.random.default_rng(5)
    vx0, vy0 = rng.normal(0.0, 30.0, count), rng.normal(0.0, 30.0, count)
    tr = lpt.Tracker(n, "fp64", sort_interval=2, sort_tile=8, tile_records=1200)
    tr.set_time_mode("pingpong")
    tr.set_snapshot(0, 0.0, ua, va)
    tr.set_snapshot(1, dt, ub, vb)
    sid = tr.add_species("inertial", 0.02, scheme, x0, y0, vx0, vy0)
    tr.step(10, dt)
    xw, yw, xu, yu = tr.get_positions(sid)
    vx, vy = tr.get_velocities(sid)
    tr.close()
    fl = oracle.grid_flow(ua, va, ub, vb, scheme=scheme, time_mode=oracle.PINGPONG)
    sp = oracle.Species(x0, y0, kind=oracle.INERTIAL, st=0.02, vx0=vx0, vy0=vy0)
    oracle.run(fl, sp, 10, dt)
    assert np.max(pdist(xw, sp.xw)) < 1e-10 and np.max(pdist(yw, sp.yw)) < 1e-10
    assert np.max(np.abs(xu - (x0 + sp.dx))) < 1e-10
    assert np.max(np.abs(yu - (y0 + sp.dy))) < 1e-10
    assert np.max(np.abs(vx - sp.vx)) < 1e-8 and np.max(np.abs(vy - sp.vy)) < 1e-8


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("scheme", ["catmull_rom", "bspline"])
def test_compat_edge_in_tiles_matches_oracle(precision, scheme):
    """The bilinear fallback near the grid edge, stencils read from the tile: the
    bounds of rounding over 12 steps (1e-10; 1e-6 in binary32 cells against the
    oracle on the rounded fields)."""
    print(f"compat edge in tiles {precision} {scheme}", flush=True)
    n, dt, count, steps = 48, 0.004, 2000, 12
    fields = synth.spectrum_snapshots(n, 5, 31, dt)
    x0, y0 = oracle.init_uniform(61, count)
    tr = lpt.Tracker(n, precision, compat_edge=True, sort_interval=4, sort_tile=8,
                     tile_records=1200)
    tr.set_time_mode("pingpong")
    tr.set_snapshot(0, 0.0, *fields[0])
    tr.set_snapshot(1, dt, *fields[1])
    a = tr.add_species("tracer", 0.0, scheme, x0, y0)
    b = tr.add_species("inertial", 0.05, scheme, x0, y0)
    tr.step(steps, dt)
    pa, pb = tr.get_positions(a), tr.get_positions(b)
    tr.close()
    if precision == "fp32_split":
        fields = [[f.astype(np.float32).astype(np.float64) for f in lv] for lv in fields]
    fl = oracle.grid_flow(*fields[0], *fields[1], scheme=scheme, time_mode=oracle.PINGPONG,
                          compat_edge=1)
    tra = oracle.Species(x0, y0)
    oracle.run(fl, tra, steps, dt)
    u0, v0 = oracle.velocity(fl, x0, y0, 0.0, step=0, t_n=0.0, dt=dt)
    ine = oracle.Species(x0, y0, kind=oracle.INERTIAL, st=0.05, vx0=u0, vy0=v0)
    oracle.run(fl, ine, steps, dt)
    tol = 1e-6 if precision == "fp32_split" else 1e-10
    for got, ref in ((pa, tra), (pb, ine)):
        assert np.max(pdist(got[0], ref.xw)) < tol and np.max(pdist(got[1], ref.yw)) < tol


def _mixed(precision, **kw):
    n, dt = 128, 0.002
    (ua, va), (ub, vb) = synth.spectrum_snapshots(n, 8, 12, dt)
    tr = lpt.Tracker(n, precision, **kw)
    tr.set_time_mode("pingpong")
    tr.set_snapshot(0, 0.0, ua, va)
    tr.set_snapshot(1, dt, ub, vb)
    sids = []
    for k, (kind, st, sch, cnt) in enumerate((("tracer", 0.0, "bilinear", 9000),
                                              ("inertial", 0.1, "catmull_rom", 4097),
                                              ("tracer", 0.0, "bspline", 65))):
        z = np.zeros(cnt)
        sids.append(tr.add_species(kind, st, sch, z, z))
        tr.init_uniform(sids[-1], 50 + k)
    return tr, sids, dt


def _snap(tr, sids):
    out = [a for s in sids for a in tr.get_positions(s)] + list(tr.get_velocities(sids[1]))
    return out + [tr.get_stats(s)[f] for s in sids for f in tr.get_stats(s).dtype.names]


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
def test_tiled_kernels_agree_over_block_sizes_and_with_the_small_ones(precision):
    """Positions, velocities and every statistics field, bit for bit: the default
    shape (small-population kernels), then tiles in blocks of 64 to 512, fused,
    interleaved and per species."""
    print(f"block sizes {precision}", flush=True)
    ref = None
    for tile, block, fused in ((0, 256, 1), (600, 64, 1), (600, 128, 2), (600, 256, 0),
                               (600, 512, 1), (-1, 256, 1)):
        tr, sids, dt = _mixed(precision, sort_interval=5, block_size=block, tile_records=tile)
        tr.set_tuning(fused=fused)
        tr.step(20, dt, stats_every=4)
        got = _snap(tr, sids)
        tr.close()
        ref = ref or got
        for a, b in zip(ref, got):
            np.testing.assert_array_equal(a, b, err_msg=f"{tile} {block} {fused}")


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
def test_graph_replays_of_tiled_runs(precision):
    """Chunks of 6 steps, which hold runs of several steps, replayed with readouts
    and synchronisations in between, against eager steps of the same kernels."""
    print(f"graph replays of tiled runs {precision}", flush=True)
    eager, sids, dt = _mixed(precision, sort_interval=8, tile_records=600)
    graph, _, _ = _mixed(precision, sort_interval=8, tile_records=600)
    graph.set_tuning(graph_chunk=6)
    for rnd, steps in enumerate((6, 12, 5, 18, 24, 6)):
        eager.step(steps, dt, stats_every=24)
        graph.step(steps, dt, stats_every=24)
        graph.synchronize()
        for a, b in zip(_snap(eager, sids), _snap(graph, sids)):
            np.testing.assert_array_equal(a, b, err_msg=f"round {rnd}")
    assert graph.get_time() == eager.get_time()
    eager.close()
    graph.close()
