"""How a generation step is divided over workgroups, looked at without a GPU."""
import glob
import os

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_18121_amd", "csrc")


def test_workgroups_exchange_at_device_scope():
    """Words that pass between workgroups are no business of a workgroup alone: a compiler may drop or merge accesses of that scope."""
    for path in glob.glob(os.path.join(CSRC, "*")):
        text = open(path).read()
        assert "HIP_MEMORY_SCOPE_WORKGROUP" not in text and "HIP_MEMORY_SCOPE_WAVEFRONT" not in text, path
