"""Sums handed from one workgroup to another inside a launch (the chunks of a heavy density tile): in the code that
the compiler makes, every wavefront waits for its write-through stores before the barrier behind which
one thread counts them as done.  A barrier waits for no stores by itself, and a fence only for those of
the wavefront that makes it."""
import re
import shutil
import subprocess

import pytest

from paper_2403_09070_amd import build


def test_write_through_stores_are_waited_for_before_the_barrier(tmp_path):
    if not shutil.which(build.HIPCC):
        pytest.skip("no hipcc")
    asm = tmp_path / "density.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", f"{build.CSRC}/density.hip", "-o", str(asm)],
                   check=True, capture_output=True)
    kernel, open_store, stores = None, None, 0
    for n, line in enumerate(asm.read_text().splitlines(), 1):
        label = re.match(r"(_Z\w+):", line)
        if label:
            kernel, open_store = label.group(1), None
        elif re.search(r"\bglobal_store_dwordx2\b.*\bsc1\b", line):
            open_store, stores = n, stores + 1
        elif re.search(r"\bs_waitcnt\b.*\bvmcnt\(0\)", line):
            open_store = None
        elif re.search(r"\bs_barrier\b", line):
            assert open_store is None, f"{kernel}: line {open_store} is in flight at the barrier of line {n}"
    assert stores >= 8, "two levels of sums in each of the four density kernels"
