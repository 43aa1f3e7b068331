"""The step kernel that bench.py names and hashes is the one that runs, the small-matrix
variant of the LDS-staged kernel included."""


def test_bench_names_the_kernel_that_runs():
    import bench

    class Stub:
        def __init__(self, kind, small):
            self.chebfd_step_kernel = lambda M, n_b: kind
            self.chebfd_step_kernel_small = lambda M, n_b: small

    names = [bench.STEP_KERNELS[bench.step_kernel(Stub(k, s), None, 32)][0]
             for k, s in ((0, False), (0, True), (1, False), (2, False), (3, False))]
    assert names == ["cheb_lds", "cheb_wave", "cheb_row", "cheb_step", "cheb_win"]
    assert all(len(bench.kernel_source_hash(k)) == 16 for k in bench.STEP_KERNELS)
