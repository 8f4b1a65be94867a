"""The bytes that bench.py's field workloads divide by, per kind of transform (no
GPU): the library's own fuse the row passes, so the step that is timed moves the
14 band spectra and, per call, the velocity; only a step whose row passes meet on
the grid moves the four grid fields twice."""
import bench


def test_built_in_transforms_move_spectra_and_one_velocity_a_call():
    n = 2048
    spec = n * 683 * 16   # the columns inside the 2/3 band: 3 * 682 < 2048 <= 3 * 683
    assert bench.ns_builtin_bytes_per_step(n, 100) == 14 * spec + 2 * n * n * 8 / 100
    assert bench.ns_field_bytes(n, 100, True) == bench.ns_builtin_bytes_per_step(n, 100)
    assert bench.ns_field_bytes(n, 100, False) == bench.ns_alg_bytes_per_step(n)


def test_coupled_step_counts_the_field_step_it_takes():
    """A coupled step calls the producer for one step at a time."""
    n, m = 2048, 1 << 20
    field = bench.ns_builtin_bytes_per_step(n, 1)
    assert (bench.coupled_alg_bytes_per_step(n, m, field)
            == bench.coupled_alg_bytes_per_step(n, m) - bench.ns_alg_bytes_per_step(n) + field)
