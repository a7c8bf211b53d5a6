"""How the FP64 residuals of several lattices are split into launches, recorded on the host
(tests/resid_table_driver.cpp): every entry's partial sums, one per 256 sites, lie in the array of the
launch without overlap, also for lattices of more than 33.5 million sites, whose sums alone are more than
the other reductions take."""
import os
import shutil
import subprocess

import pytest

from paper_2109_10687_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BIG = 1 << 26  # 67 million sites

SETS = [(8 ** 4,), (8 ** 4, 16 ** 4), (BIG,), (BIG, 8 ** 4, BIG, BIG // 2, 256), (8 ** 4, BIG), (1 << 20, 1 << 20, 1 << 25),
        (16 ** 4,) * 16, (1 << 24,) * 5, (BIG + 256 * 77, BIG)]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    if shutil.which(B.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("resid") / "driver"
    flags = [f for f in B.FLAGS if f not in ("-O3", "-Xarch_host", "-fvisibility=hidden")]
    subprocess.run([B.HIPCC] + flags + ["-O1", "-I", B.CSRC, os.path.join(ROOT, "tests", "resid_table_driver.cpp"),
                                        "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"],
                   check=True, capture_output=True, text=True)
    p = subprocess.run([str(exe)], input="".join(" ".join(map(str, s)) + "\n" for s in SETS), capture_output=True,
                       text=True, timeout=60, check=True)
    return p.stdout.splitlines()


@pytest.mark.parametrize("k", range(len(SETS)))
def test_residual_launches_hold_their_partial_sums(launches, k):
    assert "refused" not in launches[k], SETS[k]
    seen = []
    for launch in launches[k].split(";")[:-1]:
        (owner, held), ranges = (part.split() for part in launch.split(":"))
        assert int(owner) == len(seen)  # the first entry's array
        end = 0
        for r in ranges:
            first, count = map(int, r.split("+"))
            assert first == end
            end = first + count
            seen.append(count)
        assert end <= int(held), (SETS[k], launch)
    assert seen == [(v + 255) // 256 for v in SETS[k]]
