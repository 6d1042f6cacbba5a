"""Byte counts of the benchmark."""
import bench
import isdf_inputs as inp


def test_select_bytes_count_passes():
    """Every pass over the orbitals serves up to eight points where they exceed
    20 MiB (1000 k points, 52 orbitals, 40^3 grid: 53 GB), one where they do not."""
    c = inp.get_config("c5_k10_40")
    orb = c.n_k * c.n_orb * c.n_g * 16
    columns = c.n_g * 8 * (c.n_ip * (c.n_ip - 1) // 2 + 3 * c.n_ip)
    assert bench.select_bytes(c) == (c.n_ip + 7) // 8 * orb + columns
    c = inp.get_config("t_small_k2")
    assert bench.select_bytes(c) == c.n_ip * c.n_k * c.n_orb * c.n_g * 16 + c.n_g * 8 * (c.n_ip * (c.n_ip - 1) // 2 + 3 * c.n_ip)
