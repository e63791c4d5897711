"""Tilings that a plan is given and reports (host only)."""
import os
import resource
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("lmax", [0, 31, 300])
def test_pieces_longer_than_any_order(lmax):
    # in a process of its own with 4 GiB: what goes wrong takes the process along
    code = textwrap.dedent("""
        from paper_1202_6522_amd import shtn as S
        h = S.shtn_plan(%d, %d, 301, 1024)
        want = (%d // 32 + 1) * 32
        S.shtn_plan_set_tiling(h, 1, 4, 1, 1, 0, want, 0)
        ref, size = S.shtn_plan_table(h, 11).tobytes(), S.shtn_plan_device_bytes(h)
        for split in (want + 32, 1 << 20, 1 << 28, 1 << 29, 1 << 30, (1 << 31) - 32):
            S.shtn_plan_set_tiling(h, 1, 4, 1, 1, 0, split, 0)
            assert S.shtn_plan_table(h, 11).tobytes() == ref and S.shtn_plan_device_bytes(h) == size, split
            assert int(S.shtn_plan_table(h, 13)[4]) == split
        print("done")
    """ % (lmax, lmax, lmax))

    def limit():
        resource.setrlimit(resource.RLIMIT_AS, (4 << 30, 4 << 30))

    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100, preexec_fn=limit,
                       cwd=ROOT)
    assert r.returncode == 0 and "done" in r.stdout, r.stderr[-2000:]
