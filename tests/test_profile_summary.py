"""The byte counters of a profile are scaled by the copy kernel and by nothing that runs beside it."""
import json

from paper_2603_21090_amd import profile_summary


def test_traffic_is_scaled_by_the_copies_alone(tmp_path, capsys):
    names = ["layer_kernel"] * 4 + ["at::native::vectorized_elementwise_kernel<4, fill>"] + \
            ["at::native::vectorized_elementwise_kernel<4, mul>"] * 5 + ["at::native::distribution_elementwise_grid_stride_kernel"] * 4
    for counter, copy in (("FETCH_SIZE", 524_288.0), ("WRITE_SIZE", 1_048_576.0)):
        values = [10.0, 10.0, 30.0, 50.0, 7.0, 9e9] + [copy] * 4 + [1.0] * 4
        rows = [f"{i},{n.replace(',', ';')},{counter},{v}" for i, (n, v) in enumerate(zip(names, values))]
        d = tmp_path / counter
        d.mkdir()
        (d / "p_counter_collection.csv").write_text("Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value\n" + "\n".join(rows) + "\n")
    bench = {"config": {"layers": 2, "workload": "C5: a workload"}, "roofline": {"batches": [0, 1], "achieved": 1.0, "avg_launch_us": 1.0}}
    (tmp_path / "bench.json").write_text(json.dumps(bench))
    profile_summary.traffic(str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), str(tmp_path / "bench.json"))
    out = capsys.readouterr().out
    # two launches of 30 and 50 units at 2 and 1 KiB
    assert "traffic_bytes_per_launch = 122880" in out and "workload = C5" in out


def test_kernels_of_long_lists_are_layer_launches_too(tmp_path, capsys):
    names = ["layer32_kernel<2, 2, 1, 2, false>", "layer_kernel<2, 2, 1, 2, 1, 2, false, false, false>", "layer32_kernel<2, 2, 1, 2, true>"] * 2
    kernels = "".join(f'{i},"void stgn::layer_impl::{n}(args)",{2000 * i},{2000 * i + 500 + 100 * i},56,0,112,2560,0,512\n' for i, n in enumerate(names))
    (tmp_path / "p_kernel_trace.csv").write_text("Dispatch_Id,Kernel_Name,Start_Timestamp,End_Timestamp,VGPR_Count,Accum_VGPR_Count,SGPR_Count,"
                                                 "LDS_Block_Size,Scratch_Size,Workgroup_Size_X\n" + kernels)
    (tmp_path / "p_kernel_stats.csv").write_text("Name,Calls,TotalDurationNs,AverageNs,Percentage,MinNs,MaxNs\n")
    bench = {"config": {"layers": 2, "workload": "C5: a workload"},
             "roofline": {"batches": [0, 2], "achieved": 1.0, "avg_launch_us": 1.0, "event_overhead_us": 1.0, "cached_row_floats": 208}}
    (tmp_path / "bench.json").write_text(json.dumps(bench))
    profile_summary.trace(str(tmp_path), str(tmp_path / "bench.json"))
    assert "(4 launches): average 0.85 us" in capsys.readouterr().out      # 700, 800, 900 and 1,000 ns, behind the rebuild's two
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        d = tmp_path / counter
        d.mkdir()
        rows = [f"{i},{n.replace(',', ';')},{counter},{10.0 * i}" for i, n in enumerate(names)] + [f"{9 + i},vectorized_elementwise,{counter},{2.0 ** 20}" for i in range(5)]
        (d / "p_counter_collection.csv").write_text("Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value\n" + "\n".join(rows) + "\n")
    profile_summary.traffic(str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), str(tmp_path / "bench.json"))
    out = capsys.readouterr().out
    assert "4 launches: mean 35.0 units" in out and "cached_row_floats = 208" in out


def test_counter_traffic_of_another_row_width_is_not_reported(tmp_path, monkeypatch):
    import bench
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    path = tmp_path / "profiles" / "layer_kernel_C5_hbm_traffic.txt"
    path.write_text("batches = [3, 5]\ntraffic_bytes_per_launch = 100\n")
    assert bench.stored_traffic("C5", [3, 5], 208) is None                 # (a file that does not say)
    path.write_text("batches = [3, 5]\ncached_row_floats = 256\ntraffic_bytes_per_launch = 100\n")
    assert bench.stored_traffic("C5", [3, 5], 208) is None
    path.write_text("batches = [3, 5]\ncached_row_floats = 208\ntraffic_bytes_per_launch = 100\n")
    assert bench.stored_traffic("C5", [3, 5], 208) == 100.0 and bench.stored_traffic("C5", [3, 6], 208) is None
