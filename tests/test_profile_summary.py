"""Profile summaries are of one run: a directory that still holds an earlier run's files is refused, and no committed summary
lists a kernel twice or mixes builds."""
import glob
import os
import re

import pytest

from paper_2605_06534_amd import profile_summary as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STATS = '"Name","Calls","AverageNs","MinNs","MaxNs"\n"void rose::encode_kernel<0, 0, 0>(rose::EncodeArgs)",12,4.5e6,4e6,5e6\n"other()",1,1,1,1\n'
COUNTERS = ('"Dispatch_Id","Kernel_Name","Counter_Name","Counter_Value"\n1,"void rose::apply_kernel<0, 8, 8>(int)","FETCH_SIZE",10\n'
            '1,"void rose::apply_kernel<0, 8, 8>(int)","FETCH_SIZE",20\n2,"void rose::apply_kernel<0, 8, 8>(int)","FETCH_SIZE",50\n')


def put(directory, name, text):
    directory.mkdir(exist_ok=True)
    (directory / name).write_text(text)


def test_one_run(tmp_path):
    put(tmp_path / "vm", "17_kernel_stats.csv", STATS)
    put(tmp_path / "vm", "17_counter_collection.csv", COUNTERS)
    assert P.stats(str(tmp_path)) == [("encode_kernel<0,0,0>", 12, 4.5e6, 4e6, 5e6)]
    assert P.counters(str(tmp_path)) == {"apply_kernel<0,8,8>": {"FETCH_SIZE": (40.0, 2)}}


@pytest.mark.parametrize("read,name,text", [(P.stats, "kernel_stats.csv", STATS), (P.counters, "counter_collection.csv", COUNTERS)])
def test_none_or_several_runs(tmp_path, read, name, text):
    with pytest.raises(SystemExit, match="0 runs"):
        read(str(tmp_path))
    put(tmp_path / "a", "17_" + name, text)
    put(tmp_path / "b", "18_" + name, text)
    with pytest.raises(SystemExit, match="2 runs"):
        read(str(tmp_path))


def test_committed_summaries():
    builds = set()
    for path in glob.glob(os.path.join(ROOT, "profiles", "*.txt")):
        text = open(path).read()
        builds |= set(re.findall(r"kernel sources (\w+)|kernels_sha256=(\w+)", text))
        if path.endswith("_kernel_stats.txt"):
            kernels = re.findall(r"^(\w+(?:<[^>]*>)?) +\d+ +\d+ +\d+ +\d+$", text, re.M)
            assert kernels and len(kernels) == len(set(kernels)), path
    assert len({a or b for a, b in builds}) == 1
