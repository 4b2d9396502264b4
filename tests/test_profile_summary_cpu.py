"""The profile summaries read the output of one run: a directory that holds none or several is refused."""
import pytest

import bench_profile_summary as bps


@pytest.mark.parametrize("runs", [0, 1, 2])
def test_one_run_per_summary(tmp_path, runs):
    for i in range(runs):
        (tmp_path / ("host%d" % i)).mkdir()
        (tmp_path / ("host%d" % i) / "7_kernel_stats.csv").write_text("Name,Calls\nk,%d\n" % i)
        (tmp_path / ("host%d" % i) / "7_counter_collection.csv").write_text(
            "Kernel_Name,Counter_Name,Counter_Value,Dispatch_Id,Start_Timestamp,End_Timestamp\nk,C,1,1,0,9\n")
    if runs == 1:
        assert bps._only(str(tmp_path), "kernel_stats.csv").endswith("7_kernel_stats.csv")
        assert len(bps._counter_rows(str(tmp_path))) == 1
        return
    with pytest.raises(SystemExit):
        bps._counter_rows(str(tmp_path))
    with pytest.raises(SystemExit):
        bps.stats([str(tmp_path), str(tmp_path / "log"), str(tmp_path / "out.md"), "cmd"])
