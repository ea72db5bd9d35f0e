"""Calls that use the legacy stream fail while another thread captures a graph, and
break that capture: the library copies on its plans' streams only."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_17978_amd", "csrc")


def test_no_synchronous_copies():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(path) as fh:
            text = re.sub(r"//.*", "", fh.read())
        # the fill of fresh buffers that a test asks for is the one exception
        text = text.replace("(void)hipMemset(p, 0xff, bytes)", "")
        found = re.findall(r"\bhip(?:Memcpy|Memset|MemcpyDtoH|MemcpyHtoD|DeviceSynchronize)\(", text)
        assert not found, (os.path.basename(path), found)
