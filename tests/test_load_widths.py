"""The any-width condensation's listing: what is read from memory in 16-byte pieces stays in them."""
import os
import re
import subprocess

from paper_2604_12452_amd import build


def test_no_component_is_loaded_by_itself(tmp_path):
    """Rows and the summary query's piece of a lane: four bytes at a time the query alone is sixteen loads of a wavefront instead of four."""
    out = tmp_path / "condense.s"
    subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f != "-fPIC"], "-S", "--cuda-device-only", os.path.join(build.CSRC, "condense.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    kernels = re.findall(r"^(_ZN?\w*condense_any_kernel\w+):(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    assert len(kernels) == 9
    for name, listing in kernels:
        loads = re.findall(r"\t(global_load_\w+|buffer_load_\w+|flat_load_\w+)\s", listing)
        assert set(loads) == {"global_load_dwordx4"}, (name, sorted(set(loads)))
