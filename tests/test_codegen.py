"""What the compiler makes of the kernels' table reads, from the assembly of a device-only compilation (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2509_24859_amd import build


@pytest.mark.parametrize("source", ["k2_fast.hip", "k2_exact.hip"])
def test_tables_are_read_as_global_memory(source, tmp_path):
    """A flat load counts on the LDS counter too: requested early, it is waited for with the first LDS read behind it.
    A pointer that passes through inline assembly has to keep its address space for its loads not to be flat."""
    out = tmp_path / "device.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", "-w",
                           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           os.path.join(build.CSRC, source), "-o", str(out)])
    flat, kernel = {}, None
    for line in out.read_text().splitlines():
        label = re.match(r"(_Z\w+):", line)
        if label:
            kernel = label.group(1)
        elif re.match(r"\s+flat_load_", line) and re.search(r"k2_(fast|exact)", kernel):
            flat[kernel] = flat.get(kernel, 0) + 1
    assert not flat, flat
