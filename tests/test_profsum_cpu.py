"""The profile summaries on a made-up kernel trace: a single run (which has no
kernel of its own that starts it), an adjoint run whose map is scanned first, a
batch of two problems, and kernels with template arguments."""
import csv


def _trace(path, names):
    with open(path / "run_kernel_trace.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Start_Timestamp", "End_Timestamp"])
        for i, (n, us) in enumerate(names):
            w.writerow([n, 1_000_000 * i, 1_000_000 * i + 1000 * us])


TAIL = [("void (anonymous namespace)::k_walk<true, 0>(Walk, int)", 200), ("k_run_count(Walk, int)", 10),
        ("k_run_sort(Walk, int)", 10), ("void (anonymous namespace)::k_tally<16>(Walk, int)", 300),
        ("void (anonymous namespace)::k_finish<16>(Gen, Walk, int, int, int)", 100), ("k_normalise(int)", 5)]
GEN = [("k_gen_count(Gen, int)", 100), ("k_gen_scatter(Gen, int)", 100),
       ("void (anonymous namespace)::k_transport_tile<16>(Gen, int)", 800)]


def test_runs_are_cut_where_they_start(tmp_path):
    from paper_1608_05238_amd import profsum as S
    fwd = [("k_setup(ProbDev)", 5)] + GEN + TAIL
    adj = [("k_map_cdf(int)", 50), ("k_setup(ProbDev)", 5)] + GEN + GEN + TAIL
    batch = [("k_setup(ProbDev)", 5), ("k_map_cdf(int)", 50), ("k_setup(ProbDev)", 5), ("k_ctl_init(Gen)", 4)] + TAIL
    _trace(tmp_path, fwd + [("k_residual(int)", 9)] + adj + batch)
    rows = [r.split("|")[1:-1] for r in S.runs(str(tmp_path)).splitlines()[2:]]
    assert [[c.strip() for c in r] for r in rows] == [
        ["0", "8.1", "0.8", "1 / 1", "0.2", "0.2", "0.3", "0.0", "0.1"],
        ["1", "12.1", "1.6", "2 / 2", "0.4", "0.2", "0.3", "0.0", "0.1"],
        ["2", "8.1", "0.0", "0 / 0", "0.0", "0.2", "0.3", "0.0", "0.1"]]


def test_kernels_by_name_with_and_without_arguments(tmp_path):
    from paper_1608_05238_amd import profsum as S
    _trace(tmp_path, GEN + TAIL)
    assert "last 2 of 2 dispatches" in S.tail(str(tmp_path), 9, ["k_walk", "k_tally<16>"])
    assert "last 1 of 1 dispatches" in S.tail(str(tmp_path), 9, ["k_transport_tile<16>"])
