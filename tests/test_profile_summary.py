"""The summaries of profiler output count every kernel that computes a prefill linear."""
import csv
import json
import sys

import pytest

from paper_2502_00425_amd import profile_summary as ps

KERNELS = ["void (anonymous namespace)::w4a8_gemm_kernel<256, 256, 2, 4, 3, 0>(signed char const*)",
           "void (anonymous namespace)::w4a8_sliced_kernel<4, 4, 3, 0>(signed char const*)",
           "void (anonymous namespace)::w4a8_wide_kernel<4, 3, 0>(signed char const*)",
           "void (anonymous namespace)::w4a8_gemm_kernel<256, 256, 2, 4, 3, 0>(signed char const*)"]
LINEARS = ["qkv", "o", "gate_up", "down"]


def table(path, rows):
    path.parent.mkdir(exist_ok=True)
    with open(path, "w", newline="") as f:
        w = csv.DictWriter(f, rows[0].keys())
        w.writeheader()
        w.writerows(rows)


def test_labels_of_a_trace(tmp_path):
    rows = [{"Kernel_Name": k, "Workgroup_Size_X": 512, "Grid_Size_X": 512 * (10 + i % 4), "Start_Timestamp": 100000 * i,
             "End_Timestamp": 100000 * i + 1000 * (i % 4 + 1)} for i, k in enumerate(KERNELS * 2)]
    table(tmp_path / "a_kernel_trace.csv", rows)
    lines = ps.trace_table(str(tmp_path), LINEARS).splitlines()[2:]
    got = {(c[2], c[3]): (c[4], c[5]) for c in ([x.strip() for x in l.split("|")] for l in lines)}
    assert got == {(p, str(10 + i)): ("2", f"{i + 1:.2f}") for i, p in enumerate(LINEARS)}


def test_bytes_of_a_step(tmp_path, monkeypatch, capsys):
    """Two steps of four linears at 1, 2, 4 and 8 MiB each way, one of them with a split-K reduction of 16."""
    copy = "__amd_rocclr_copyBuffer.kd"
    mib = {KERNELS[0] + "a": 1, KERNELS[1]: 2, KERNELS[2]: 4, KERNELS[3] + "b": 8, "void splitk_reduce_kernel<0>(int)": 16}
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        rows = [{"Counter_Name": counter, "Dispatch_Id": 0, "Counter_Value": ps.GIB_KIB / 2, "Kernel_Name": copy, "Grid_Size": 64,
                 "Workgroup_Size": 64}]
        for step in range(2):
            rows += [{"Counter_Name": counter, "Dispatch_Id": 1 + step * 5 + i, "Counter_Value": m * 512, "Kernel_Name": k,
                      "Grid_Size": 512 * (i + 1), "Workgroup_Size": 512} for i, (k, m) in enumerate(mib.items())]
        table(tmp_path / counter / "b_counter_collection.csv", rows)
    out = tmp_path / "t.json"
    monkeypatch.setattr(sys, "argv", ["x", "--config", "1", "--fetch", str(tmp_path / "FETCH_SIZE"), "--write",
                                      str(tmp_path / "WRITE_SIZE"), "--steps", "2", "--build-id", "b", "--json", str(out)])
    ps.main()
    c = json.loads(out.read_text())["configs"]["c1"]
    assert c["gemm_launches_counted"] == 8
    assert c["kernels"] == ["w4a8_gemm_kernel", "w4a8_sliced_kernel", "w4a8_wide_kernel"]
    assert c["bytes_per_step"] == pytest.approx(2 * 31 * 2 ** 20) and c["bytes_per_gemm_launch"] == pytest.approx(2 * 31 * 2 ** 18)
