"""bench.py looks kernels up by name in the committed byte-counter summaries: the names are those of the present sources."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kernel_names_of_the_bench_exist_and_are_found_in_the_summaries():
    import bench
    csrc = "".join(open(f).read() for f in glob.glob(os.path.join(ROOT, "paper_2508_18224_amd", "csrc", "*.hip")))
    kernels = set(re.findall(r"__global__ void[^;{]*?\b(k_\w+)\(", csrc))
    named = {n for names in bench.KERNEL_NAMES.values() for n in names} | set(bench.NOT_IN_STEP)
    assert {n.replace("nsa::", "") for n in named} <= kernels, named
    summaries = glob.glob(os.path.join(ROOT, "profiles", "hot_path_*.txt"))
    assert summaries
    for path in summaries:
        workload = os.path.basename(path)[len("hot_path_"):-len(".txt")]
        traffic, _ = bench.measured_traffic(workload)
        for kind in ("fwd_main", "bwd_main", "bwd_delta", "bwd_dq_reduce"):
            assert any(n in traffic for n in bench.KERNEL_NAMES[kind]), (path, kind)
        # every kernel a summary gives bytes for is one of the sources'
        assert {n.replace("nsa::", "") for n in traffic} <= kernels, (path, traffic)
