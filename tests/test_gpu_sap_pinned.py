"""The packed-FP16 SAP bit for bit against pinned results (golden/sap_fp16.txt).

In half precision a last-bit change of the FP32 sums of the face hop terms moves a block's scale and with
it every rounding after it: 1e-3 of the result, as large as its whole error, so no tolerance can tell such
a change from the rounding itself.  The pinned digests are those of the half-sweep whose sums take each
term in one fused multiply-add.  The inputs are made from integers by single IEEE operations (products,
sums, a division, a square root), so they are the same on every machine.
"""
import hashlib
import os

import numpy as np
import pytest
import torch

import paper_2109_10687_amd as dd

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "sap_fp16.txt")
PHASES = (1.0, complex(0.6, 0.8), -1.0, complex(0.0, 1.0))


def integers(n, salt):
    """n integers -8 .. 8 (a multiplicative hash of their index)."""
    i = np.arange(n, dtype=np.uint64) + np.uint64(salt) * np.uint64(1000003)
    h = (i * np.uint64(0x9E3779B97F4A7C15)) ^ (i >> np.uint64(3))
    h = h * np.uint64(0xBF58476D1CE4E5B9)
    return ((h >> np.uint64(40)) % np.uint64(17)).astype(np.float64) - 8.0


def links(dims, salt):
    """SU(3) links, each the product of an SU(2) rotation of rows 0, 1 and one of rows 1, 2."""
    n = 4 * int(np.prod(dims))
    q = []
    for k in range(2):
        v = integers(4 * n, salt + k).reshape(n, 4)
        v[:, 0] = 16.0 + v[:, 0]  # near the unit matrix
        q.append(v / np.sqrt(v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1] + (v[:, 2] * v[:, 2] + v[:, 3] * v[:, 3]))[:, None])

    def mul(ar, ai, br, bi):
        return ar * br - ai * bi, ar * bi + ai * br

    a, b = (q[0][:, 0], q[0][:, 1]), (q[0][:, 2], q[0][:, 3])
    c, d = (q[1][:, 0], q[1][:, 1]), (q[1][:, 2], q[1][:, 3])
    zero = (np.zeros(n), np.zeros(n))
    conj = lambda z: (z[0], -z[1])
    neg = lambda z: (-z[0], -z[1])
    rows = [[a, mul(*b, *c), mul(*b, *d)], [neg(conj(b)), mul(*conj(a), *c), mul(*conj(a), *d)],
            [zero, neg(conj(d)), conj(c)]]
    U = np.empty((n, 3, 3, 2))
    for r in range(3):
        for s in range(3):
            U[:, r, s, 0], U[:, r, s, 1] = rows[r][s]
    return torch.view_as_complex(torch.from_numpy(U)).reshape((4,) + tuple(reversed(dims)) + (3, 3))


def spinor(dims, salt):
    x = integers(24 * int(np.prod(dims)), salt).reshape(tuple(reversed(dims)) + (3, 4, 2)) + 0.125
    return torch.view_as_complex(torch.from_numpy(x))


def digest(t):
    return hashlib.sha256(t.cpu().numpy().tobytes()).hexdigest()[:16]


def pinned():
    out = []
    for line in open(GOLDEN):
        if not line.startswith("#"):
            *shape, n_sap, n_jac, one, batch = line.split()
            out.append((tuple(map(int, shape[:4])), tuple(map(int, shape[4:])), int(n_sap), int(n_jac), one, batch))
    return out


@pytest.mark.parametrize("dims, block, n_sap, n_jac, one, batch", pinned())
def test_packed_fp16_sap_bits(dims, block, n_sap, n_jac, one, batch):
    s = dd.Solver(dd.Params(dims=dims, kappa=0.13, csw=1.0, block=block, phases=PHASES, n_sap=n_sap, n_jac=n_jac),
                  links(dims, 1).cuda())
    x = spinor(dims, 7).cuda()
    got = digest(s.precondition(x, prec=dd.DD_F16)), digest(s.precondition_batch(torch.stack([x, x.flip(0)])))
    s.close()
    assert got == (one, batch), got
