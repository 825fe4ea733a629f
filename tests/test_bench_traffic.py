"""bench.py reports counter figures of a profile only for the code that they were taken of (CPU only)."""
import shutil

from test_bench_formulas import bench  # noqa: F401  (fixture: imports bench.py)

NAME = "pf::scan_kernel<128, 64, 32, 16, true, false>"


def test_traffic_belongs_to_the_profiled_code(bench):  # noqa: F811
    table = {"code_digest": "abc", "cfg4": {"scan_kernel": {"name": NAME, "bytes": 7}}}
    assert bench.profiled_traffic(table, "cfg4", "scan_kernel", NAME, "abc") == 7
    assert bench.profiled_traffic(table, "cfg4", "scan_kernel", NAME, "abd") is None             # other code, same name
    assert bench.profiled_traffic(table, "cfg4", "scan_kernel", NAME[:-6] + "true>", "abc") is None
    assert bench.profiled_traffic(table, "cfg2", "scan_kernel", NAME, "abc") is None
    assert bench.profiled_traffic({"cfg4": table["cfg4"]}, "cfg4", "scan_kernel", NAME, "abc") is None   # code not recorded


def test_digest_follows_the_code_and_nothing_else(bench, tmp_path):  # noqa: F811
    import os
    csrc = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_2504_00492_amd", "csrc")
    copy = tmp_path / "csrc"
    shutil.copytree(csrc, copy, ignore=shutil.ignore_patterns("*.o"))
    digest = bench.kernel_code_digest()
    assert bench.kernel_code_digest(str(copy)) == digest
    chain = copy / "pf_chain.h"
    text = chain.read_text()
    chain.write_text("// a remark\n" + text.replace("\n", "\n\n") + "/* another\n one */\n")
    assert bench.kernel_code_digest(str(copy)) == digest
    chain.write_text(text.replace("fit < 6 ? fit : 6", "fit < 4 ? fit : 4"))
    assert bench.kernel_code_digest(str(copy)) != digest


def test_launch_times_need_the_described_launches(bench):  # noqa: F811
    names = ["pf::flow_kernel<64, 64, 64, false>", "pf::scan_kernel<64, 64, 64, 16, true, false>"]
    trace = [(10, names[0], 2.0), (13, names[1], 5.0), (30, names[1], 7.0), (20, names[0], 4.0)]
    assert bench.launch_times(trace, names) == [3.0, 6.0]
    assert bench.launch_times(trace[:3], names) is None                     # a launch is missing
    assert bench.launch_times(trace, names[:1]) is None                     # one that is not described
    assert bench.launch_times(trace + [(40, names[1], 1.0), (41, names[0], 1.0)], names) is None   # another order
    assert bench.launch_times([], names) is None and bench.launch_times(trace, []) is None
