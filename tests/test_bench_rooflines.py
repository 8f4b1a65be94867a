"""What bench.py's rooflines name and divide by (no GPU).  The field workloads
count the bytes of the transforms in use: the built-in ones fuse the row passes, so
the step that is timed moves the 14 band spectra and, per call, the velocity; only a
step whose row passes meet on the grid moves the four grid fields twice."""
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


def test_step_kernel_names_follow_the_route():
    """Small populations in the default launch shape run their own kernels."""
    from paper_2607_17836_amd import workloads
    assert bench.step_kernel_name(workloads.C1_TG) == "small64_kernel<bilinear, tracers>"
    assert bench.step_kernel_name(workloads.C1_TG, dict(sort_interval=20, fused=1)).startswith("small")
    assert bench.step_kernel_name(workloads.C1_TG, dict(persistent=1)).startswith("step64")
    assert bench.step_kernel_name(workloads.C3_SPLIT) == "step32_kernel<bilinear, tracers>"
