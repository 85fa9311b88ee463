"""The profile summaries' selection of kernels by name."""
import csv
import os
import re

from paper_2211_01185_amd import build, counter_summary, pmc_summary


def _name(*args):
    return f"void cfddem::force_kick<{', '.join(args)}>(cfddem::Dev, int, int, int const*, int)"


def test_force_kernel_patterns_match_the_kernels_of_this_source():
    with open(os.path.join(build.CSRC, "dem_kernels.hip")) as fh:
        sig = re.search(r"template <([^>]*)>\s*__global__[^;{]*?void force_kick\(", fh.read()).group(1)
    assert [p.split()[-1] for p in sig.split(",")] == ["R", "ADVANCE", "CONT", "L", "ROLL", "S"]
    prime, step = pmc_summary.force_kernel_names(2)
    assert prime.search(_name("float", "false", "false", "2", "false", "4"))
    for cont in ("true", "false"):
        assert step.search(_name("float", "true", cont, "2", "false", "1"))
        assert not step.search(_name("float", "true", cont, "2", "true", "1"))  # rolling friction
        assert not step.search(_name("float", "true", cont, "4", "false", "1"))
        assert not step.search(_name("double", "true", cont, "2", "false", "1"))
    assert not prime.search(_name("float", "true", "true", "2", "false", "1"))


def test_region_takes_the_steps_of_the_last_bed(tmp_path):
    prime, step = _name("float", "false", "false", "2", "false", "1"), _name("float", "true", "true", "2", "false", "1")
    kernels = [prime, step, step, prime, "other", step, step, "other", step]
    with open(tmp_path / "1_counter_collection.csv", "w", newline="") as fh:
        w = csv.DictWriter(fh, ["Dispatch_Id", "Counter_Name", "Kernel_Name", "Counter_Value"])
        w.writeheader()
        for i, k in enumerate(kernels):
            w.writerow(dict(Dispatch_Id=i, Counter_Name="C", Kernel_Name=k, Counter_Value=i))
    assert pmc_summary._region(str(tmp_path), "C", 2, 1, 2) == [6.0, 8.0]
    assert counter_summary._region is pmc_summary._region
