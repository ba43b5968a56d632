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
