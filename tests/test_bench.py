"""bench.py's bookkeeping: which kernels a counter run is summed over, and which kernel the roofline is quoted for (no GPU)."""
import json
import os

import pytest

import bench


def counter_csv(directory, counter, readings):
    directory.mkdir(parents=True)
    with open(directory / "pmc_counter_collection.csv", "w") as f:
        f.write('"Kernel_Name","Counter_Name","Counter_Value"\n')
        for name, value in readings:
            f.write(f'"{name}","{counter}",{value}\n')


def record(tmp_path, monkeypatch, kernels):
    for what, counter in (("fetch", "FETCH_SIZE"), ("write", "WRITE_SIZE")):
        counter_csv(tmp_path / ("cal_" + what), counter, [("copy", 1 << 20), ("copy", 1 << 20)])        # KiB: 1 GiB, scale 1
        counter_csv(tmp_path / what, counter, [(name, kib) for name, kib in kernels for _ in range(2)])
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "traffic.json"))
    bench.record_traffic(str(tmp_path), "key")
    with open(tmp_path / "traffic.json") as f:
        return json.load(f)["entries"]["key"]


@pytest.mark.parametrize("kernel", ["void (anonymous namespace)::spmm_gather_kernel<_Float16, 128>(SpmmArgs)",
                                    "void (anonymous namespace)::spmm_task_kernel_f32<128>(SpmmArgs)"])
def test_traffic_is_that_of_the_task_kernel_and_the_clearing_kernel(tmp_path, monkeypatch, kernel):
    e = record(tmp_path, monkeypatch, [(kernel, 300), ("zero_rows_kernel(int const*, long)", 20), ("sddmm_task_kernel<_Float16, 32, 1, true>", 7000)])
    assert e["fetch_bytes"] == e["write_bytes"] == 320 * 1024 and e["bytes"] == 640 * 1024


def test_a_counter_run_without_the_task_kernel_is_refused(tmp_path, monkeypatch):
    with pytest.raises(SystemExit):
        record(tmp_path, monkeypatch, [("zero_rows_kernel(int const*, long)", 20)])


def test_the_kernel_that_the_roofline_names_is_one_of_the_library():
    assert bench.spmm_kernel_name("f16", 128) == "spmm_gather_kernel<f16,128>"
    assert bench.spmm_kernel_name("bf16", 224) == "spmm_gather_kernel<bf16,128>"        # wide operands run in pieces of 128 columns
    assert bench.spmm_kernel_name("f16", 96) == "spmm_gather_kernel<f16,64>"
    assert bench.spmm_kernel_name("f32", 48) == "spmm_task_kernel_f32<32>"
    with open(os.path.join(bench.SOURCE_DIRS[0], "kernels.hip")) as f:
        source = f.read()
    for name in bench.SPMM_TASK_KERNELS + ("zero_rows_kernel",):
        assert f"void {name}(" in source, name
