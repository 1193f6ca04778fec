"""The peaks that bench.py holds the edge kernels against."""
import bench


def test_matrix_peak_counts_the_terms_of_every_product():
    """F = 64: 8192 flops in the F x F product, 1024 in one with the eight basis functions; the forward kernel has one of
    these, the reverse kernel two, always as six terms."""
    assert bench.flops_fwd_edge(64) == 9216 and bench.flops_bwd_edge_as_defined(64) == 10240
    for precision, terms in (("f32", 6), ("f32split", 3), ("bf16", 1)):
        assert abs(bench.matrix_peak_tflops(precision, 64, 1) - 2500 * 9216 / (8192 * terms + 1024 * 6)) < 1e-9
        assert abs(bench.matrix_peak_tflops(precision, 64, 2) - 2500 * 10240 / (8192 * terms + 2048 * 6)) < 1e-9
    assert abs(bench.matrix_peak_tflops("f32", 64, 2) - 2500 / 6) < 1e-9
