"""What the LDS race check (tests/test_gpu_racecheck.py) relies on in the sources: every function that
declares LDS shared by several wavefronts waits at entry (wg_skew), before its first store to it, and has
its barriers through wg_barrier, which waits as well.  Kernels of one wavefront per workgroup
share nothing."""
import glob
import os
import re

from paper_2109_10687_amd import build as B


def functions():
    """(name, whether it is a kernel of 64 threads, body) of every function that declares LDS."""
    for path in sorted(glob.glob(os.path.join(B.CSRC, "*.hip")) + glob.glob(os.path.join(B.CSRC, "*.h"))):
        src = re.sub(r"//.*", "", open(path).read())
        # __launch_bounds__(256, 2) -> threads_256, __launch_bounds__(64 * TT, 2) -> threads_many
        src = re.sub(r"__launch_bounds__\(\s*([^,()]*?)\s*(?:,[^()]*)?\)",
                     lambda m: "threads_" + (m.group(1) if m.group(1).isdigit() else "many"), src)
        for m in re.finditer(r"^((?:__global__|DD_INL|template)[^;{}]*?)\b(\w+)\s*\(([^;{}]*)\)\s*\{", src, re.M):
            depth, k = 1, m.end()
            while depth:
                depth += {"{": 1, "}": -1}.get(src[k], 0)
                k += 1
            body = src[m.end():k]
            if "__shared__" in body:
                yield m.group(2), "threads_64 " in m.group(1), body


def test_functions_that_share_lds_wait_at_entry():
    found = list(functions())
    names = {n for n, _, _ in found}
    assert {"k_dirac_can", "k_dirac_ts", "k_sap_half", "sap_half_pk_body", "finalize_sum", "wg_reduce_store_at",
            "k_dirac_rhs_res", "k_pack_spinor"} <= names, names
    for name, one_wavefront, body in found:
        assert "__syncthreads" not in body, name
        if one_wavefront:
            continue
        barrier = min(body.find(w) for w in ("wg_barrier", "sap_barrier") if w in body)
        assert 0 <= body.find("wg_skew()") < barrier, name
