"""What the benchmark line says of a search workload: the kernels that run and the bytes that
cannot be done without, for fused and unfused searches (no GPU)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_kernel_names():
    assert bench.forward_kernel("direct", "u8") == "direct_u8_kernel"
    assert bench.forward_kernel("direct", "f32") == "direct_f32_kernel"
    assert bench.forward_kernel("u8m_q4_dpw4_nw8_cc4_row2304_buf2", "u8") == "u8m_kernel"
    assert bench.forward_kernel("u8s_q4_dpw4_nw16_cc4_o8", "u8") == "u8s_kernel"
    assert bench.forward_kernel("u8_q4_dpw4_nw4_cc16_buf1", "u8") == "u8_kernel"
    assert bench.forward_kernel("lane_q1_dpw1_nw8_cc8_row384_ring4", "f32") == "lane_kernel"
    unfused = bench.search_kernels("unfused", "win_tp20_dpw4_nw16_win40_cc10_buf2_jmp", "f32")
    assert unfused.startswith("win_kernel + ") and "stored series" in unfused and "epilogue" not in unfused
    assert bench.search_kernels("unfused", "u8m_x", "u8").startswith("u8m_kernel + ")
    assert bench.search_kernels("u8m_x", "u8s_y", "u8") == "u8m_det_kernel with the search epilogue + det_finish_kernel"
    assert bench.search_kernels("win_x", "lane_y", "f32") == "win_kernel with the search epilogue + det_finish_kernel"


def test_search_bytes_leave_the_series_out():
    # 1024 channels x 20,100 samples and 2000 DM trials: 82.3 MB of input, 8.2 MB of delays, 64 KB of results
    assert bench.search_bytes(1024, 2000, 20100, 4, 0) == 1024 * 20100 * 4 + 4 * 1024 * 2000 + 32 * 2000
    assert bench.search_bytes(32, 2048, 200100, 1, 1 << 20) - bench.search_bytes(32, 2048, 200100, 1, 0) == 1 << 20
