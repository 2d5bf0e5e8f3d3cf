"""The kernel groups of profile_summary.py are named as the library's kernels are."""
import re
import shutil
import subprocess

import pytest

from paper_2511_04283_amd import build
from paper_2511_04283_amd import profile_summary as P


@pytest.mark.skipif(not shutil.which("nm"), reason="no nm")
def test_every_prefix_of_a_group_is_that_of_a_kernel():
    """A prefix that no kernel has leaves its group without traffic, and nothing says so."""
    symbols = subprocess.run(["nm", "-C", build.LIB], check=True, capture_output=True, text=True).stdout
    kernels = {P.short(line.split(" ", 2)[2].replace("__device_stub__", "")) for line in symbols.splitlines() if re.search(r"\bk_\w+|__device_stub__", line)}
    for group, prefixes in P.GROUPS.items():
        for prefix in prefixes:
            assert any(k.startswith(prefix) for k in kernels), (group, prefix)
