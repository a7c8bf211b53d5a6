"""The launch of the half-sweep that several lattices share, recorded on the host
(tests/sap_multi_launch_driver.cpp): workgroups, threads and LDS must not depend on the order in
which the caller lists its lattices, and the LDS must leave room for the three workgroups per CU that the
kernel's registers allow (160 KB)."""
import itertools
import os
import shutil
import subprocess

import pytest

from paper_2109_10687_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    if shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("launch") / "driver"
    flags = [f for f in B.FLAGS if f not in ("-O3", "-Xarch_host", "-fvisibility=hidden")]
    subprocess.run([B.HIPCC] + flags + ["-O1", "-I", B.CSRC, os.path.join(ROOT, "tests", "sap_multi_launch_driver.cpp"),
                                        "-o", str(exe)], check=True, capture_output=True, text=True)

    def run(groups):
        lines = "".join(" ".join(f"{a} {b} {c} {d}" for a, b, c, d in g) + "\n" for g in groups)
        p = subprocess.run([str(exe)], input=lines, capture_output=True, text=True, timeout=60, check=True)
        out = []
        for line in p.stdout.splitlines():
            out.append("refused" if "refused" in line else
                       [tuple(map(int, line.split()[k:k + 3])) for k in range(0, len(line.split()), 3)])
        return out

    return run


def test_shared_half_sweep_is_launched_alike_in_every_order(launches):
    b4, b2, odd = (4, 4, 4, 4), (2, 2, 2, 2), (4, 2, 4, 2)
    orders = sorted(set(itertools.permutations((b4, b4, b2, b2))))
    got = launches(orders)
    assert got[0] == [(2 * 128 + 2 * 8, 256, got[0][0][2])]
    assert all(g == got[0] for g in got), dict(zip(orders, got))
    for group in (orders[0], (b4,), (b2,), (odd, odd)):
        (wgs, threads, lds), = launches([group])[0]
        assert 3 * lds <= 160 * 1024, (group, wgs, threads, lds)
    assert launches([(b4, odd)]) == ["refused"]
    # more lattices than a table holds: several launches
    assert len(launches([(b2, b4) * 7])[0]) == 2
