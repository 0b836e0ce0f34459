"""Kernel names that qspec_describe_kernel gives: the symbol that is launched and that a profiler reports, and its place in the
tables that benchmark and profile summary build from such symbols.  Needs no GPU."""
import pytest

import bench
import profile_summary
from paper_2410_11305_amd import binding as B


def mangled(name):
    """Head of the symbol of "namespace::kernel<bool, int, int>" in namespace qspec."""
    *spaces, rest = ("qspec::" + name).split("::")
    kernel, args = rest.rstrip(">").split("<")
    value = {"true": "Lb1E", "false": "Lb0E"}
    return "_ZN" + "".join(f"{len(s)}{s}" for s in spaces + [kernel]) + "I" + "".join(value.get(a, f"Li{a}E") for a in args.split(", ")) + "E"


@pytest.mark.parametrize("draft", [True, False])
@pytest.mark.parametrize("M,nt", [(5, 2), (16, 6), (17, 2), (32, 4)])
def test_streaming_plans_name_the_kernel_of_their_wavefronts(plan, draft, M, nt):
    code = open(B.LIB_PATH, "rb").read()
    names = []
    for waves in (8, 4):
        plan("QSPEC_STREAM_W4A4" if draft else "QSPEC_STREAM_W4A16", f"{nt},1,1,{waves}")
        names.append(B.describe_kernel(draft, M, 4096, 4096))
        assert mangled(names[-1]).encode() in code
    assert names[1] == "waves4::" + names[0] and names[0].startswith("gemm_stream_kernel<")
    family = names[0].rsplit(", ", 1)[0] + ", *>"
    for name in names:
        assert bench.family(name) == family
        symbol = f"void qspec::{name}(uint4 const*, unsigned short const*, int) [clone .kd]"
        assert profile_summary._short(symbol) == name and profile_summary._family(name) == family


def test_the_profile_summary_keeps_both(tmp_path):
    names = ["gemm_stream_kernel<true, 1, 2>", "waves4::gemm_stream_kernel<true, 1, 2>"]
    with open(tmp_path / "kt_kernel_stats.csv", "w") as f:
        f.write('"Name","Calls","TotalDurationNs","AverageNs","Percentage","MinNs","MaxNs"\n')
        for n in names:
            f.write(f'"void qspec::{n}(int)",3,30000,10000,50.0,9000,11000\n')
    for counter in ("fetch", "write"):
        with open(tmp_path / f"{counter}_counter_collection.csv", "w") as f:
            f.write('"Kernel_Name","Counter_Name","Counter_Value"\n"__amd_rocclr_copyBuffer","C",262144\n')
            for n in names:
                f.write(f'"void qspec::{n}(int)","C",1024\n')
    profile_summary.main(str(tmp_path), str(tmp_path / "out"), "t2")
    stats = (tmp_path / "out" / "t2_kernel_stats.txt").read_text()
    assert all(f"  {n} " in stats for n in names) and "gemm_stream_kernel<true, 1, *> " in stats and stats.count("*>") == 1
    assert all(n in (tmp_path / "out" / "t2_hbm_counters.txt").read_text() for n in names)
