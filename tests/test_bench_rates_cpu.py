"""The rates that bench.py derives from the library's per-kernel bytes."""
import bench


def test_variable_coefficient_rates_count_the_bytes_read():
    """Each pass counts 32 bytes of face conductivities an unknown and reads 16:
    24 + 16 of stencil_dot, 96 + 16 of pcg_pass; a pass without bytes has no rate."""
    dof = 1000
    stats = {"stencil_dot": dict(launches=4, seconds=2e-6, bytes=4 * 56 * dof),
             "pcg_pass": dict(launches=3, seconds=3e-6, bytes=3 * 128 * dof),
             "final_check": dict(launches=1, seconds=1e-6, bytes=0)}
    t = bench.vc_kern_table(stats, dof)
    assert t["stencil_dot"]["GBps"] == round(4 * 40 * dof / 2e-6 / 1e9, 1)
    assert t["pcg_pass"]["GBps"] == round(3 * 112 * dof / 3e-6 / 1e9, 1)
    assert t["final_check"]["GBps"] == 0.0
