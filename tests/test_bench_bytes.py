"""Algorithmic bytes of the benchmark's triangle product."""
import bench


def test_triangle_bytes_count_what_a_group_shares():
    # no entries: signs and 16-bit y of 64 probes a row, and 5/16 of the row pointer
    assert bench.triangle_bytes(1000, 0) == 136 * 1000 + 5 / 16 * 4 * 1001
    # 16 entries a row: 5/16 of their 64 bytes more
    assert bench.triangle_bytes(1000, 16000) - bench.triangle_bytes(1000, 0) == 5 / 16 * 64000
