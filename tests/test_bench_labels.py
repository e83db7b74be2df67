"""The benchmark line names the kernel that runs: the fused pass's form differs by
precision at the headline grid."""


def test_the_dominant_kernel_is_named_by_its_form():
    import bench
    ms = {"x_fwd": 0.3, "z_fwd": 2.7, "y_fused": 7.5, "z_inv": 2.8, "x_inv": 2.9, "finalize": 0.1}
    for prec, kernel in (("fp64", "k_fused_wide"), ("fp32", "k_fused")):
        r = bench.summarize(prec, 20, 0.025, ms, {"energy": 1.0})
        assert r["roofline"]["pass"] == "y_fused" and r["roofline"]["kernel"] == kernel
