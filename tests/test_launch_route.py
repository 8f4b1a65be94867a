"""Which step kernels a context launches (no GPU needed): the small-population
kernels only while the launch shape is the default one, so that a tile, a halo, a
workgroup cap, rows or species launches that a caller asks for take effect."""
import pytest

import hip_stand_in

SCRIPT = r"""
precision, count, kw = sys.argv[2], int(sys.argv[3]), eval(sys.argv[4])
n, schemes = kw.pop("n", 16), kw.pop("schemes", ("bilinear", "catmull_rom"))
tr = lpt.Tracker(n, precision, tile_records=kw.pop("created_with", 0))
u = np.zeros((n, n))
tr.set_snapshot(0, 0.0, u, u)
tr.set_snapshot(1, 1.0, u, u)
x = np.linspace(0.0, 6.0, count)
for scheme in schemes:
    tr.add_species("tracer", 0.0, scheme, x, x)
tr.set_tuning(**kw)
launched()
tr.step(20, 0.01)
print(*launched())
"""

SHAPES = [dict(tile_records=-1), dict(tile_records=64), dict(created_with=800),
          dict(persistent=1, max_workgroups=8), dict(rows=2, block_size=512), dict(fused=0),
          dict(fused=2), dict(halo_scale=0.5)]
DEFAULTS = [dict(), dict(block_size=64), dict(halo_scale=0.125, fused=1, rows=1, persistent=0),
            dict(sort_interval=3, sort_cells=0), dict(max_workgroups=8)]


def _kernels(tmp_path, precision, count, kw):
    names = hip_stand_in.run(SCRIPT, tmp_path, precision, count, kw).split()
    steps = [n for n in names if any(k in n for k in ("small", "run", "step")) and
             "kernel" in n and "fin_" not in n]
    assert steps
    return steps


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("kw", SHAPES)
def test_an_asked_for_shape_takes_the_tiled_kernels(tmp_path, precision, kw):
    for name in _kernels(tmp_path, precision, 1000, dict(kw)):
        assert "run64_kernel" in name or "run32_kernel" in name, name


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
@pytest.mark.parametrize("kw", DEFAULTS)
def test_the_default_shape_leaves_small_populations_to_their_kernels(tmp_path, precision, kw):
    for name in _kernels(tmp_path, precision, 1000, dict(kw)):
        assert "small64_kernel" in name or "small32_kernel" in name, name
    for name in _kernels(tmp_path, precision, 1 << 19, dict(kw)):
        assert "small" not in name, name


@pytest.mark.parametrize("precision,scheme,n,count,small", [
    ("fp64", "bilinear", 2048, 1 << 19, True),         # n^2 / 8
    ("fp64", "bilinear", 2048, (1 << 19) + 1, False),
    ("fp64", "bilinear", 3500, 3500 * 3500 // 8, True),
    ("fp64", "bilinear", 4096, 1 << 21, False),        # n^2 / 8, too many
    ("fp64", "bilinear", 16, 1 << 18, True),
    ("fp32_split", "bilinear", 4096, 1 << 20, True),
    ("fp32_split", "bilinear", 2048, (1 << 18) + 1, False),
    ("fp64", "bspline", 1024, 1 << 16, True),          # n^2 / 16
    ("fp64", "bspline", 1024, (1 << 16) + 1, False)])
def test_the_population_line(tmp_path, precision, scheme, n, count, small):
    for name in _kernels(tmp_path, precision, count, dict(n=n, schemes=(scheme,))):
        assert ("small" in name) == small, name
