"""The benchmark's roofline reports the HBM traffic that the counters of the
GEMM kernel gave; the figure holds only for the sources it was taken with."""
import bench


def test_stored_traffic_is_of_the_current_gemm_sources():
    assert bench.measured_traffic("w4a4_linear") is not None
