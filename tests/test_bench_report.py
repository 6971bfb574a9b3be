"""The benchmark's report of a job's inner loops (host arithmetic only)."""
import bench


def test_loops_that_stop_early_are_credited_with_what_they_ran():
    """Six inner loops of three modes, every record timed: the passes are the ones
    computed, the compulsory bytes count once per loop, whether a loop gave one
    record (row by row) or one per pass (Phi launches)."""
    N, R, nnz, dims, segs = 3, 4, 1_000, [30, 20, 10], [30, 20, 10]
    minb = 2 * sum(bench.phi_min_bytes(N, R, nnz, dims, segs, n) for n in range(N))
    st = dict(phi_evals=6 * 3, outer_iters=2)  # stopped at the third of lmax passes
    whole = [(n % N, 3.0) for n in range(6)]
    single = [(n % N, 1.0) for n in range(6) for _ in range(3)]
    for recs in (whole, single):
        roof, rep = bench.loop_report(N, R, nnz, dims, segs, 8, recs, 1, 1, st, 20.0)
        assert rep["avg_ms"] == 1.0 and rep["passes_per_step"] == 18 and rep["loops_per_step"] == 6
        assert rep["nnz_per_s"] == 1e6 and rep["share_of_step"] == 18.0 / 20.0
        assert roof["achieved"] == minb / 18e-3 / 1e9
    half = [(n % N, 3.0) for n in (0, 2, 4)]  # every second record
    assert bench.loop_report(N, R, nnz, dims, segs, 8, half, 2, 1, st, 20.0)[1]["avg_ms"] == 1.0
