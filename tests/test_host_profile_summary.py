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
        for prefix in (alternative for p in prefixes for alternative in (p if isinstance(p, tuple) else (p,))):
            assert any(k.startswith(prefix) for k in kernels), (group, prefix)


def test_of_alternatives_the_first_that_ran_counts():
    render = P.GROUPS["render_fwd"]
    with_record, without = "k_render_fwd<true, true, true>", "k_render_fwd<true, true, false>"
    assert P.group_total({with_record: 5.0, without: 3.0, "k_render_fwd<false, true, false>": 9.0}, render) == 5.0
    assert P.group_total({without: 3.0}, render) == 3.0
    assert P.group_total({"k_preprocess<3, false, false>": 9.0}, render) == 0.0
    assert P.group_total({"k_tile_layout": 2.0, "k_tile_pairs<false, false, false>": 1.0}, P.GROUPS["emit_pairs"]) == 3.0
