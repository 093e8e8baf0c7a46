"""A step's launchers allocate nothing on the host and cannot throw through the C
entries (acat.h: the functions never abort or throw): no strings or containers of the
standard library in the launch code.  The kernel timer, off by default, keeps its records
in acat_profile.cpp; acat_batch_init builds its tables in acat_api.hip."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2007_01416_amd", "csrc")


def test_no_allocating_types_in_launch_code():
    files = [f for f in glob.glob(os.path.join(CSRC, "*")) if f.endswith((".hip", ".hpp"))]
    assert len(files) >= 10
    for f in files:
        if os.path.basename(f) == "acat_api.hip":
            continue
        text = open(f).read()
        found = re.findall(r"std::(?:string|to_string|vector|map|function|unique_ptr|shared_ptr)\b", text)
        assert not found, (os.path.basename(f), found)
