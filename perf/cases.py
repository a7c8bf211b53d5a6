"""What this framework is asked to do, as cases that can be timed and checked.

Every case is work that a lattice-QCD program has the library do through its Python entry points:
the Dirac operator by itself (measurements, residuals), the operator and the Schwarz preconditioner
as the parts of a Krylov solver of one's own, the mixed-precision solves for one source, for the
twelve point sources of a propagator and for several lattices, the fermion force of molecular
dynamics, and the loss |D^-1 phi|^2 with its gradients.  Lattices run from 8^4 (one launch is the
whole cost) to 48^3 x 96 (one field is over half a gigabyte); 4^4 blocks are the usual ones, 2^4
blocks serve extents that are no multiple of 8.

Results come back at the precision that they have: single-precision ones as FP32 fields in the
library's own layout, the half-precision preconditioner's rounded to half precision, the others as
canonical complex128 tensors.  `exact` works the same quantities out in 64 bits with plain
torch on the canonical fields.
"""
import math

import torch

import paper_2109_10687_amd as dd
from paper_2109_10687_amd.autograd import quark_loss

PHASES = (1.0, 1.0, 1.0, -1.0)   # periodic in space, antiperiodic in time

# the uneven set of lattices of the several-lattice workload: (dims, block side)
MULTI = (((8, 8, 8, 8), 4), ((8, 8, 8, 8), 4), ((12, 12, 12, 12), 2), ((12, 12, 12, 12), 2),
         ((16, 16, 16, 16), 4), ((16, 16, 16, 16), 4), ((16, 16, 16, 32), 4), ((16, 16, 16, 32), 4))


def _dims(text):
    return tuple(int(v) for v in text.split("x"))


def _shape(dims):
    return tuple(reversed(dims))


def _volume(dims):
    return math.prod(dims)


# ---------------------------------------------------------------------------------- the cases

def listed():
    return [
        # smallest call: the operator on a test-sized lattice, all launch and call overhead
        {"name": "dirac_f64_8x8x8x8", "do": "dirac_f64", "op": "D", "dims": "8x8x8x8", "block": 4, "kappa": 0.1365, "csw": 1.7},
        # the FP64 residual of a source on an ordinary lattice
        {"name": "dirac_f64_24x24x24x48", "do": "dirac_f64", "op": "D", "dims": "24x24x24x48", "block": 4, "kappa": 0.1365, "csw": 1.7},
        # uneven extents, which only 2^4 blocks divide, and the adjoint operator
        {"name": "ddag_f64_12x20x28x36", "do": "dirac_f64", "op": "Ddag", "dims": "12x20x28x36", "block": 2, "kappa": 0.12, "csw": 1.0},
        # the FP32 operator inside a Krylov loop on the propagator lattice
        {"name": "dirac_f32_32x32x32x64", "do": "dirac_f32", "dims": "32x32x32x64", "block": 4, "kappa": 0.133, "csw": 1.7},
        # the inner solver's operator (FP16-stored input) on the largest lattice
        {"name": "dirac_f16in_48x48x48x96", "do": "dirac_f16in", "dims": "48x48x48x96", "block": 4, "kappa": 0.133, "csw": 1.7},
        # the preconditioner in half and in single precision
        {"name": "sap_f16_32x32x32x32", "do": "sap", "prec": "f16", "dims": "32x32x32x32", "block": 4, "kappa": 0.1365, "csw": 1.7, "n_sap": 6, "n_jac": 4},
        {"name": "sap_f32_16x16x24x32", "do": "sap", "prec": "f32", "dims": "16x16x24x32", "block": 4, "kappa": 0.1365, "csw": 1.7, "n_sap": 4, "n_jac": 4},
        # molecular dynamics: the su(3) force
        {"name": "force_24x24x24x24", "do": "force", "su3": True, "dims": "24x24x24x24", "block": 4, "kappa": 0.133, "csw": 1.7},
        # whole calls: one source, the twelve point sources of a propagator, eight lattices at once
        {"name": "solve_32x32x32x64", "do": "solve", "mode": "mixed", "dims": "32x32x32x64", "block": 4, "kappa": 0.133, "csw": 1.7, "n_sap": 6},
        {"name": "propagator_16x16x16x32", "do": "batch", "nrhs": 12, "dims": "16x16x16x32", "block": 4, "kappa": 0.13, "csw": 1.7, "n_sap": 6},
        {"name": "multi_8_lattices", "do": "multi", "nlat": 8, "kappa": 0.13, "csw": 1.7, "n_sap": 6},
        # a training step: new links, forward and adjoint solve, gradients of links, source and c_SW
        {"name": "loss_16x16x16x16", "do": "loss", "dims": "16x16x16x16", "block": 4, "kappa": 0.125, "csw": 1.7, "n_sap": 4},
    ]


def _draw_dims(rng, block, lo, hi):
    """Extents that are multiples of two blocks, their volume spread evenly over its logarithm."""
    step = 2 * block
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    while True:
        side = want ** 0.25
        d = [max(1, round(side * math.exp(rng.uniform(-0.4, 0.4)) / step)) * step for _ in range(4)]
        if 0.6 * lo <= math.prod(d) <= hi:
            return "x".join(str(v) for v in d)


def draw(rng):
    do = rng.choice(["dirac_f64", "dirac_f64", "dirac_f32", "dirac_f16in", "sap", "sap", "force", "solve", "batch", "multi", "loss"])
    block = rng.choice([4, 4, 4, 2])
    c = {"do": do, "block": block, "kappa": round(rng.uniform(0.11, 0.13), 4), "csw": round(rng.uniform(1.0, 1.7), 3)}
    if do == "dirac_f64":
        c.update(op=rng.choice(["D", "D", "Ddag"]), dims=_draw_dims(rng, block, 4096, 24 ** 3 * 48))
    elif do in ("dirac_f32", "dirac_f16in"):
        c.update(dims=_draw_dims(rng, block, 4096, 32 ** 3 * 64))
    elif do == "sap":
        c.update(prec=rng.choice(["f16", "f16", "f32"]), dims=_draw_dims(rng, block, 4096, 32 ** 4), n_sap=rng.choice([2, 4, 6]), n_jac=rng.choice([4, 4, 3, 5]))
    elif do == "force":
        c.update(su3=rng.choice([True, False]), dims=_draw_dims(rng, block, 4096, 24 ** 4))
    elif do == "solve":
        c.update(mode=rng.choice(["mixed", "mixed", "fgmres", "plain"]), dims=_draw_dims(rng, block, 4096, 24 ** 3 * 48), n_sap=rng.choice([4, 6]))
    elif do == "batch":
        c.update(nrhs=rng.choice([2, 3, 5, 8, 12]), dims=_draw_dims(rng, block, 4096, 16 ** 3 * 32), n_sap=rng.choice([4, 6]))
    elif do == "multi":
        c.update(nlat=rng.randint(2, 8), n_sap=rng.choice([4, 6]))
        del c["block"]
    else:
        c.update(dims=_draw_dims(rng, block, 4096, 16 ** 4), n_sap=rng.choice([4, 6]))
    return c


# ---------------------------------------------------------------------------------- inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _mul3(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _links(dims, gen, eps=0.3):
    """Random SU(3) links exp(i eps H), H Hermitian with Gaussian entries (plaquette near 0.6)."""
    n = 4 * _volume(dims)
    out = torch.empty((n, 3, 3), dtype=torch.complex128, device="cuda")
    eye = torch.eye(3, dtype=torch.complex128, device="cuda")
    for lo in range(0, n, 1 << 20):
        m = min(1 << 20, n - lo)
        z = torch.view_as_complex(torch.randn((m, 3, 3, 2), generator=gen, dtype=torch.float64, device="cuda"))
        x = 0.5j * eps * (z + z.conj().transpose(-1, -2))
        u = eye + x / 12
        for k in range(11, 0, -1):
            u = eye + _mul3(x, u) / k
        # what the series leaves open: orthonormal rows; and the trace of H: the third row of an SU(3) matrix
        a = u[:, 0] / torch.linalg.vector_norm(u[:, 0], dim=-1, keepdim=True)
        b = u[:, 1] - (a.conj() * u[:, 1]).sum(-1, keepdim=True) * a
        b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
        out[lo:lo + m] = torch.stack((a, b, torch.linalg.cross(a, b).conj()), dim=1)
    return out.reshape((4,) + _shape(dims) + (3, 3))


def _gaussian(dims, gen):
    return torch.view_as_complex(torch.randn(_shape(dims) + (3, 4, 2), generator=gen, dtype=torch.float64, device="cuda"))


def _point_sources(dims, nrhs, seed):
    """The first nrhs of the twelve spin-colour unit vectors at one site (another site for another seed)."""
    g = torch.Generator()
    g.manual_seed(int(seed) + 1)
    x, y, z, t = (int(torch.randint(0, n, (1,), generator=g)) for n in dims)
    b = torch.zeros((nrhs,) + _shape(dims) + (3, 4), dtype=torch.complex128, device="cuda")
    for r in range(nrhs):
        b[r, t, z, y, x, r // 4, r % 4] = 1.0
    return b


def _params(case, dims, block):
    return dd.Params(dims=dims, kappa=case["kappa"], csw=case["csw"], block=(block,) * 4, phases=PHASES,
                     n_sap=case.get("n_sap", 4), n_jac=case.get("n_jac", 4))


def _inputs(case, seed):
    """The fields of a case, in the order they are drawn."""
    gen = _generator(seed)
    if case["do"] == "multi":
        lats = MULTI[-case["nlat"]:]
        return [(_links(d, gen), _gaussian(d, gen)) for d, _ in lats]
    dims = _dims(case["dims"])
    U = _links(dims, gen)
    if case["do"] == "batch":
        return U, _point_sources(dims, case["nrhs"], seed)
    if case["do"] == "force":
        return U, _gaussian(dims, gen), _gaussian(dims, gen)
    return U, _gaussian(dims, gen)


TOL = 1e-12   # of the solves: forces and gradients are taken from them


def prepare(case, seed):
    do = case["do"]
    if do == "multi":
        lats = MULTI[-case["nlat"]:]
        m = dd.Multi([_params(case, d, b) for d, b in lats])
        fields = _inputs(case, seed)
        for k, (U, _) in enumerate(fields):
            m.load_gauge(k, U)
        return {"do": do, "multi": m, "b": [b for _, b in fields]}
    dims = _dims(case["dims"])
    U, *fields = _inputs(case, seed)
    s = dd.Solver(_params(case, dims, case["block"]), None if do == "loss" else U)
    st = {"do": do, "case": dict(case), "solver": s, "in": fields, "values": 24 * _volume(dims)}
    if do == "dirac_f32":
        st["x"], st["q"] = s.pack(fields[0], dd.DD_F32), s.field(dd.DD_F32)
    elif do == "dirac_f16in":
        st["x"], st["q"] = s.pack(fields[0], dd.DD_F16), s.field(dd.DD_F32)
    elif do == "sap":
        st["z"], st["zf"] = s.new_spinor(), s.field(dd.DD_F32)
    elif do == "loss":
        st["U"] = U
        st["csw"] = torch.tensor(case["csw"], dtype=torch.float64)
    elif do == "solve":
        st["mode"] = {"mixed": dd.DD_SOLVE_MIXED, "fgmres": dd.DD_SOLVE_FGMRES, "plain": dd.DD_SOLVE_F64_PLAIN}[case["mode"]]
    if do in ("dirac_f32", "dirac_f16in"):
        del st["in"]
    return st


# ---------------------------------------------------------------------------------- one pass

def _f32(st, field):
    """An FP32 field of the library as its numbers."""
    return field[:4 * st["values"]].view(torch.float32)


def _converged(infos):
    for i in infos:
        if i["status"] != "DD_OK":
            raise RuntimeError(f"solve: {i}")


def run(st):
    do = st["do"]
    if do == "multi":
        xs, infos = st["multi"].solve(st["b"], tol=TOL)
        _converged(infos)
        return xs
    s, case = st["solver"], st["case"]
    if do == "dirac_f64":
        return s.apply(st["in"][0], op=dd.DD_OP_D if case["op"] == "D" else dd.DD_OP_DDAG, prec=dd.DD_F64)
    if do == "dirac_f32":
        return _f32(st, s.apply_packed(st["q"], st["x"], op=dd.DD_OP_A, prec=dd.DD_F32))
    if do == "dirac_f16in":
        return _f32(st, s.apply_packed_f16in(st["q"], st["x"]))
    if do == "sap":
        if case["prec"] == "f16":
            # z = M_SAP r to half precision, which is what a program keeps of it
            return torch.view_as_real(s.precondition(st["in"][0], prec=dd.DD_F16, out=st["z"])).to(torch.float16)
        # z = M_SAP r, then into the FP32 field that a Krylov loop goes on with
        s.precondition(st["in"][0], prec=dd.DD_F32, out=st["z"])
        return _f32(st, s.pack(st["z"], dd.DD_F32, out=st["zf"]))
    if do == "force":
        force, dcsw = s.force(st["in"][0], st["in"][1], su3=case["su3"])
        return {"force": force, "dcsw": dcsw}
    if do == "solve":
        x, info = s.solve(st["in"][0], tol=TOL, mode=st["mode"])
        _converged([info])
        return x
    if do == "batch":
        x, infos = s.solve_batch(st["in"][0], tol=TOL)
        _converged(infos)
        return x
    U = st["U"].detach().requires_grad_()
    phi = st["in"][0].detach().requires_grad_()
    csw = st["csw"].detach().requires_grad_()
    loss = quark_loss(U, phi, csw, s, tol=TOL)
    loss.backward()
    return {"loss": loss.detach(), "U": U.grad, "phi": phi.grad, "csw": csw.grad}


# ---------------------------------------------------------------------------------- what a pass needs

HOPS = 6 * 168 + 2 * 156   # flops of the eight hops of a site
CLOVER = 600               # flops of the two 6x6 Hermitian blocks
LINKS64, CLOVER64 = 576, 576
LINKS32, CLOVER32 = 192, 288   # FP32 with two rows of a link; half of it in FP16


def work(case):
    do = case["do"]
    if do == "multi":
        V = sum(_volume(d) for d, _ in MULTI[-case["nlat"]:])
        return {"bytes": V * (192 * 2 + LINKS64 + CLOVER64), "flops": V * (HOPS + CLOVER)}
    V = _volume(_dims(case["dims"]))
    if do == "dirac_f64":
        return {"bytes": V * (192 * 2 + LINKS64 + CLOVER64), "flops": V * (HOPS + CLOVER)}
    if do == "dirac_f32":
        return {"bytes": V * (96 * 2 + LINKS32 + CLOVER32), "flops": V * (HOPS + CLOVER)}
    if do == "dirac_f16in":
        return {"bytes": V * (52 + 96 + LINKS32 + CLOVER32), "flops": V * (HOPS + CLOVER)}
    if do == "sap":
        # the source read, the result written, links and clover read once; every site takes n_sap + 1
        # block solves of n_jac in-block operators (3/4 of the hops), and the cross-block rest in between
        half = 2 if case["prec"] == "f16" else 1
        solves = (case["n_sap"] + 1) * case["n_jac"] * (0.75 * HOPS + CLOVER)
        return {"bytes": V * (192 + 96 + (LINKS32 + CLOVER32) // half), "flops": V * (solves + case["n_sap"] * (HOPS + CLOVER))}
    if do == "force":
        return {"bytes": V * (2 * 192 + 2 * LINKS64 + CLOVER64), "flops": V * 44592}
    n = case.get("nrhs", 1)
    if do in ("solve", "batch"):
        # at the least one residual; how many iterations a solve takes is not known beforehand
        return {"bytes": V * (n * 2 * 192 + LINKS64 + CLOVER64), "flops": n * V * (HOPS + CLOVER)}
    return {"bytes": V * (4 * 192 + 2 * LINKS64 + 2 * CLOVER64), "flops": V * (2 * (HOPS + CLOVER) + 44592)}


# ---------------------------------------------------------------------------------- the same in 64 bits

# gamma_1..gamma_4 (Dirac representation, gamma_4 diagonal): (gamma psi)_a = f_a psi_(p_a)
GAMMA = (((3, 2, 1, 0), (1j, 1j, -1j, -1j)), ((3, 2, 1, 0), (1, -1, -1, 1)),
         ((2, 3, 0, 1), (1j, -1j, -1j, 1j)), ((0, 1, 2, 3), (1, 1, -1, -1)))


def _gamma(mu, x):
    p, f = GAMMA[mu]
    return x[..., list(p)] * torch.tensor(f, dtype=x.dtype, device=x.device)


def _dag(u):
    return u.conj().transpose(-1, -2)


def _colour(u, x):
    return (u.unsqueeze(-1) * x.unsqueeze(-3)).sum(-2)


def _hopping(U, x, lead):
    """sum_mu (1 - gamma_mu) U_mu(n) x(n + mu) + (1 + gamma_mu) U_mu(n - mu)^dagger x(n - mu); U carries the phases."""
    y = torch.zeros_like(x)
    for mu in range(4):
        d = lead + 3 - mu
        f = _colour(U[mu], torch.roll(x, -1, d))
        b = torch.roll(_colour(_dag(U[mu]), x), 1, d)
        y = y + (f + b) - _gamma(mu, f - b)
    return y


def _with_phases(U):
    out = []
    for mu in range(4):
        d = 3 - mu
        ph = torch.ones(U.shape[1 + d], dtype=U.dtype, device=U.device)
        ph[-1] = PHASES[mu]
        out.append(U[mu] * ph.reshape([-1 if k == d else 1 for k in range(6)]))
    return out


def _field_strength(U):
    """{(mu, nu): F}: (Q - Q^dagger) / 8 of the four plaquettes in the plane that start and end at the site."""
    F = {}
    for mu in range(4):
        for nu in range(mu + 1, 4):
            def at(k, a, b, mu=mu, nu=nu):   # U_k(n + a mu + b nu)
                v = U[k]
                v = torch.roll(v, -a, 3 - mu) if a else v
                return torch.roll(v, -b, 3 - nu) if b else v
            Q = _mul3(_mul3(at(mu, 0, 0), at(nu, 1, 0)), _dag(_mul3(at(nu, 0, 0), at(mu, 0, 1))))
            Q = Q + _mul3(_mul3(at(nu, 0, 0), _dag(at(mu, -1, 1))), _mul3(_dag(at(nu, -1, 0)), at(mu, -1, 0)))
            Q = Q + _mul3(_dag(_mul3(at(nu, -1, -1), at(mu, -1, 0))), _mul3(at(mu, -1, -1), at(nu, 0, -1)))
            Q = Q + _mul3(_mul3(_dag(at(nu, 0, -1)), at(mu, 0, -1)), _mul3(at(nu, 1, -1), _dag(at(mu, 0, 0))))
            F[mu, nu] = (Q - _dag(Q)) / 8
    return F


def _clover(F, x, kappa):
    """(C / c_SW) x = i kappa sum_(mu < nu) sigma F x with sigma = i gamma_mu gamma_nu."""
    y = torch.zeros_like(x)
    for (mu, nu), f in F.items():
        y = y - kappa * _colour(f, _gamma(mu, _gamma(nu, x)))
    return y


class _Operator:
    def __init__(self, case, U, inverse=False):
        self.kappa, self.csw = case["kappa"], case["csw"]
        self.U, self.F = _with_phases(U), _field_strength(U)
        if inverse:
            self.inv = self._inverse()

    def D(self, x, lead=0):
        return x + self.csw * _clover(self.F, x, self.kappa) - self.kappa * _hopping(self.U, x, lead)

    def Ddag(self, x, lead=0):
        g5 = [2, 3, 0, 1]
        return self.D(x[..., g5], lead)[..., g5]

    def _inverse(self):
        """(1 + C)^-1 per site as 12 x 12 matrices: Gauss-Jordan, the matrix is positive definite."""
        shape = self.U[0].shape[:4]
        n = math.prod(shape)
        out = torch.empty((n, 12, 12), dtype=torch.complex128, device="cuda")
        Fs = {k: f.reshape(n, 3, 3) for k, f in self.F.items()}
        unit = torch.eye(12, dtype=torch.complex128, device="cuda").reshape(12, 3, 4)
        for lo in range(0, n, 1 << 18):
            part = {k: f[lo:lo + (1 << 18), None] for k, f in Fs.items()}
            m = next(iter(part.values())).shape[0]
            e = unit.expand(m, 12, 3, 4)
            M = (e + self.csw * _clover(part, e, self.kappa)).reshape(m, 12, 12).transpose(1, 2).contiguous()
            for k in range(12):
                p = 1 / M[:, k, k].clone()
                row, col = M[:, k, :] * p[:, None], M[:, :, k].clone()
                row[:, k] = p
                M[:, :, k] = 0
                M[:, k, :] = 0
                col[:, k] = -1
                M -= col[:, :, None] * row[:, None, :]
            out[lo:lo + m] = M
        return out

    def solve_clover(self, x):
        n = self.inv.shape[0]
        v, out = x.reshape(n, 1, 12), torch.empty((n, 12), dtype=x.dtype, device=x.device)
        for lo in range(0, n, 1 << 20):
            out[lo:lo + (1 << 20)] = (self.inv[lo:lo + (1 << 20)] * v[lo:lo + (1 << 20)]).sum(-1)
        return out.reshape(x.shape)

    def A(self, x, U=None):
        return x - self.kappa * self.solve_clover(_hopping(self.U if U is None else U, x, 0))

    def sap(self, b, block, n_sap, n_jac):
        """sum_(j <= n_sap) K (1 - A K)^j b, K the two-colour block sweep with n_jac Jacobi steps per block."""
        inside, colour = [], 0
        for mu in range(4):
            d = 3 - mu
            c = torch.arange(b.shape[d], device="cuda").reshape([-1 if k == d else 1 for k in range(4)])
            inside.append(self.U[mu] * (c % block != block - 1)[..., None, None])
            colour = colour + c // block
        even = (colour % 2 == 0)[..., None, None]

        def solve_blocks(v):
            acc = r = v
            for _ in range(n_jac):
                r = r - self.A(r, inside)
                acc = acc + r
            return acc

        s, x = b, torch.zeros_like(b)
        for j in range(n_sap + 1):
            z = solve_blocks(s * even)
            z = z + solve_blocks((s - self.A(z)) * ~even)
            x = x + z
            if j < n_sap:
                s = s - self.A(z)
        return x

    def solve(self, b, apply, lead=0):
        """apply(x) = b to rounding: BiCGStab, restarted from the true residual; None if it does not get there."""
        def dot(u, v):
            return (u.conj() * v).flatten(lead).sum(-1).reshape((-1,) + (1,) * 6 if lead else ())
        x = torch.zeros_like(b)
        bb = dot(b, b).real
        for _ in range(3):
            r = b - apply(x)
            if bool((dot(r, r).real <= 1e-29 * bb).all()):
                break
            start = dot(r, r).real.clamp_min(1e-300)
            r0, p, y, rho = r, r, torch.zeros_like(b), dot(r, r)
            live = torch.ones_like(start, dtype=torch.bool)
            for _ in range(2000):
                q = apply(p)
                a = rho / dot(r0, q)
                s = r - a * q
                t = apply(s)
                w = dot(t, s) / dot(t, t)
                y = torch.where(live, y + a * p + w * s, y)
                r = torch.where(live, s - w * t, r)
                live = live & (dot(r, r).real > 1e-20 * start)
                if not bool(live.any()):
                    break
                rho, old = dot(r0, r), rho
                p = r + (rho / old) * (a / w) * (p - w * q)
                p = torch.where(live, p, r0)
            x = x + y
        r = b - apply(x)
        return x if bool((dot(r, r).real <= 1e-27 * bb).all()) else None


def _gradients(case, U, psi, chi):
    """d/dU of -2 Re <chi| D(U) psi> (as dL/dRe U + i dL/dIm U) and d/dc_SW of it."""
    U = U.detach().requires_grad_()
    csw = torch.tensor(case["csw"], dtype=torch.float64, device="cuda", requires_grad=True)
    op = _Operator(dict(case, csw=csw), U)
    (-2 * (chi.conj() * op.D(psi)).sum().real).backward()
    return U.grad, float(csw.grad)


def _exact_force(case, seed):
    U, psi, chi = _inputs(case, seed)
    G, dcsw = _gradients(case, U, psi, chi)
    if case["su3"]:
        X = _mul3(U, _dag(G))
        H = 0.5j * (X - _dag(X))
        tr = H.diagonal(dim1=-2, dim2=-1).sum(-1) / 3
        G = H - tr[..., None, None] * torch.eye(3, dtype=H.dtype, device="cuda")
    return {"force": G, "dcsw": dcsw}


def _block_major(x, block):
    """A canonical spinor in the library's order of an FP32 field: blocks, (spin, colour), sites of the block."""
    t, z, y, w = (n // block for n in x.shape[:4])
    v = x.reshape(t, block, z, block, y, block, w, block, 3, 4)
    return torch.view_as_real(v.permute(0, 2, 4, 6, 9, 8, 1, 3, 5, 7).contiguous()).reshape(-1)


def exact(case, seed):
    do = case["do"]
    if do == "multi":
        lats = MULTI[-case["nlat"]:]
        out = []
        for (U, b), _ in zip(_inputs(case, seed), lats):
            op = _Operator(case, U)
            out.append(op.solve(b, op.D))
        return out
    if do == "force":
        return _exact_force(case, seed)
    U, b = _inputs(case, seed)
    if do == "dirac_f64":
        op = _Operator(case, U)
        return op.D(b) if case["op"] == "D" else op.Ddag(b)
    if do in ("dirac_f32", "dirac_f16in"):
        return _block_major(_Operator(case, U, inverse=True).A(b), case["block"])
    if do == "sap":
        z = _Operator(case, U, inverse=True).sap(b, case["block"], case["n_sap"], case["n_jac"])
        return torch.view_as_real(z) if case["prec"] == "f16" else _block_major(z, case["block"])
    op = _Operator(case, U)
    if do == "solve":
        # on the largest lattices plain torch takes too long for it
        return op.solve(b, op.D) if _volume(_dims(case["dims"])) <= 24 ** 3 * 48 else None
    if do == "batch":
        return op.solve(b, lambda x: op.D(x, 1), lead=1)
    psi = op.solve(b, op.D)
    chi = op.solve(psi, op.Ddag)
    G, dcsw = _gradients(case, U, psi, chi)
    return {"loss": (psi.conj() * psi).sum().real, "U": G, "phi": 2 * chi, "csw": torch.tensor(dcsw, dtype=torch.float64)}
