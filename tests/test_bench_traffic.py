"""Which of a profiled run's launches bench.py takes the kernel's HBM traffic from."""
from bench import traffic_launches


def test_only_the_timed_launches_count():
    timed, clocked = "wfst_channel_kernel2<true, false, false, false, true>(x)", "wfst_channel_kernel2<true, false, true, false, true>(x)"
    run = [("probe_copy(x)", 1.0), (timed, 10.0), (timed, 20.0), (timed, 22.0), (clocked, 90.0), ("probe_copy(x)", 3.0)]
    rows = [{"Dispatch_Id": str(7 + i), "Kernel_Name": k, "Counter_Name": c, "Counter_Value": str(v + (c != "FETCH_SIZE"))}
            for i, (k, v) in enumerate(run) for c in ("FETCH_SIZE", "WRITE_SIZE")]
    assert traffic_launches(rows, "FETCH_SIZE", 2) == ([20.0, 22.0], [1.0, 3.0])
    assert traffic_launches(rows[::-1], "WRITE_SIZE", 2) == ([21.0, 23.0], [2.0, 4.0])
    assert traffic_launches([], "FETCH_SIZE", 2) == ([], [])
