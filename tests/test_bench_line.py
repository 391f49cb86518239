"""The benchmark's dense-LU rate: given where the trailing-update record says that a dense LU ran, whatever its speed."""
import bench


def test_dense_rate_follows_the_gemm_record():
    lu = 64 * (8.0 / 3.0) * 1000.0 ** 3
    assert bench._dense_tflops(lu, 1.0, 0.01 * lu) is None  # a slow structured operator: its border's GEMMs
    assert bench._dense_tflops(lu, 1.0, 0.0) is None
    assert bench._dense_tflops(lu, 1e-4, 0.8 * lu) == lu / 1e-4 / 1e12  # a dense one, also above the peak
    assert bench._dense_tflops(lu, 0.0, 0.8 * lu) is None
