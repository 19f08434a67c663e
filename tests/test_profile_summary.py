"""The traffic file that bench.py reads, from counter runs: the kernels it names are those of the library, and a
renamed one is an error, not a missing figure."""

import json
import sqlite3
import subprocess

import pytest

from paper_2411_15100_amd import profile_summary as ps
from paper_2411_15100_amd.binding import _LIB_PATH


def _library_kernels():
    out = subprocess.run(["nm", "-C", _LIB_PATH], capture_output=True, text=True, check=True).stdout
    return sorted({line.split(" ", 2)[2] for line in out.splitlines() if "_kernel" in line and " d " in line and "xgm::" in line})


def _counter_run(path, counter, kernels):
    db = sqlite3.connect(path)
    db.execute("create table counters_collection (kernel_name text, counter_name text, value real)")
    copy = "void at::native::vectorized_elementwise_kernel<4, at::native::bfloat16_copy_kernel_cuda(at::TensorIteratorBase&)>(int)"
    values = {copy: 38000.0} | {k: 10.0 + n for n, k in enumerate(kernels)}
    db.executemany("insert into counters_collection values (?, ?, ?)", [(k, counter, v) for k, v in values.items() for _ in range(3)])
    db.commit()
    db.close()
    return values


def test_traffic_of_the_librarys_kernels(tmp_path):
    kernels = _library_kernels()
    assert len(kernels) > 20
    runs, values = [], {}
    for label, counter in (("fetch", "FETCH_SIZE"), ("write", "WRITE_SIZE")):
        values[counter] = _counter_run(tmp_path / label, counter, kernels)
        runs.append((label, str(tmp_path / label)))
    ps.counters(str(tmp_path / "out.txt"), str(tmp_path / "traffic.json"), "note", runs)
    traffic = json.load(open(tmp_path / "traffic.json"))
    assert traffic["kernel_source_hash"] == ps.kernel_source_hash()
    assert set(traffic["bytes_per_launch"]) == set(ps.STEP_KERNELS.values())
    for name, total in traffic["bytes_per_launch"].items():
        full, = [k for k in kernels if f"::{name}(" in k]
        assert total == pytest.approx((2.0 * values["FETCH_SIZE"][full] + values["WRITE_SIZE"][full]) * 1024.0)
    text = open(tmp_path / "out.txt").read()
    assert all(ps.short(k) in text for k in kernels)
    # a kernel of the step that no run has
    others = [k for k in kernels if f"::{ps.STEP_KERNELS['fill']}(" not in k]
    runs = []
    for label, counter in (("fetch2", "FETCH_SIZE"), ("write2", "WRITE_SIZE")):
        _counter_run(tmp_path / label, counter, others)
        runs.append((label, str(tmp_path / label)))
    with pytest.raises(SystemExit):
        ps.counters(str(tmp_path / "out2.txt"), str(tmp_path / "traffic2.json"), "note", runs)
    assert not (tmp_path / "traffic2.json").exists()
