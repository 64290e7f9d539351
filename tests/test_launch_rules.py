"""The rules that choose a launch by sizes (lbm_plan.h), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++20", "-O1", "-Wall", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2212_07494_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "launch_rules.cpp"), "-o", exe], check=True)

    def run(queries):
        text = "\n".join(" ".join(str(v) for v in q) for q in queries) + "\n"
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]

    return run


# nwaves, groups, longest group, Q, nx, rows
@pytest.mark.parametrize("query,by_node", [
    ((1, 1, 1, 27, 1, 10 ** 6), 1), ((185, 1, 185, 27, 1, 10 ** 6), 1),
    ((9, 5, 4, 19, 16, 62500), 1), ((185, 9, 42, 27, 128, 16384), 0),
    ((185, 9, 42, 27, 32, 62500), 0), ((1, 1, 1, 27, 128, 16384), 1),
    ((0, 0, 0, 9, 64, 32), 1),
    # the rows' launch would pass 2^32 threads: 2^26 rows
    ((10 ** 4, 16, 700, 39, 31, 1 << 26), 1), ((10 ** 4, 16, 700, 39, 31, 1 << 25), 0)])
def test_waves_by_node(ask, query, by_node):
    assert ask([("waves_by_node", *query)]) == [[by_node]]
