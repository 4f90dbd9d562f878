"""The byte model of the present kernels for small 1D plans, whose workgroup moves the Lanczos
vectors and the basis only."""
import bench


def test_one_workgroup_solves():
    w = bench.WORKLOADS["wave1d_63x64"]
    N = 63 * 64
    for prec in ("fp64", "fp32"):   # the scratch, of either precision, stays in LDS
        got = bench.algorithmic_bytes(w, prec, iters_total=6, solves=1, fused=True, resident=True)
        setup = 8 * N + 3 * 8 * N
        steps = 6 * (16 * N + 8 * N) + 5 * 8 * N
        check = 6 * 8 * N + 8 * N + 8 * N
        assert got == {"iter": setup + steps + check}
    one = bench.algorithmic_bytes(w, "fp64", 6, 1, fused=True, resident=True)["iter"]
    assert bench.algorithmic_bytes(w, "fp64", 60, 10, fused=True, resident=True)["iter"] == 10 * one
