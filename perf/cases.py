"""Performance cases: what users of the library have it do, with inputs, sizes and exact results.

Kinds of case (all through the Python binding, as a user's program calls it):

* ``solve``      a batch of independent Poisson problems on one uniform box mesh
                 (``Context.solve_batch``): Hartree potentials, pair potentials.
* ``exchange``   the exchange step of N orbitals (``Context.exchange``): pair densities, their
                 solves, W_k, K_ij and E_x.
* ``uneven``     one batch over three meshes of different sizes, interleaved.
* ``boundary``   Dirichlet data by quadrature of the sources (``Context.boundary_data``).
* ``octree``     right-hand sides and solves on the adaptive octree mesh (``Octree.rhs/solve``).
* ``consumers``  projected Hartree action, build and action of the compressed exchange.
* ``network``    forward and backward pass of the initial-guess network, the body of its training.

Every solve stops at the FP64 relative residual 1e-11 unless stated, the tolerance at which the
benchmark compares its arms.  Sources are Gaussian densities or products of orbitals over s
Gaussians with exponents log-uniform in [0.3, 10], with closed-form (erf) boundary data.
"""
import functools
import math
import os

import numpy as np
import torch

from paper_2510_21213_amd import binding

RTOL = 1e-11
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(binding.__file__)), "weights")


def listed():
    return [
        # one small Hartree problem, the latency of a call: 4^3 elements of degree 3
        {"name": "hartree_4e_p3", "kind": "solve", "ex": 4, "ey": 4, "ez": 4, "p": 3, "nrhs": 1, "h": 2.5,
         "precision": "fp64", "guess": False, "gl": False},
        # a few densities on a ragged box of odd degree (the general operator kernels)
        {"name": "ragged_p5", "kind": "solve", "ex": 10, "ey": 14, "ez": 12, "p": 5, "nrhs": 5, "h": 1.0,
         "precision": "fp32_pc", "guess": False, "gl": False},
        # Gauss-Legendre nodes, the paper's node family
        {"name": "gl_8e_p4", "kind": "solve", "ex": 8, "ey": 8, "ez": 8, "p": 4, "nrhs": 36, "h": 1.0,
         "precision": "fp32_pc", "guess": False, "gl": True},
        # one SCF exchange step of 8 orbitals in the mixed precision with the learned guess
        {"name": "exchange8_bf16f", "kind": "exchange", "ex": 16, "ey": 16, "ez": 16, "p": 4, "norb": 8, "h": 1.0,
         "precision": "bf16f_pc", "guess": True},
        # the same step in plain FP64
        {"name": "exchange8_fp64", "kind": "exchange", "ex": 16, "ey": 16, "ez": 16, "p": 4, "norb": 8, "h": 1.0,
         "precision": "fp64", "guess": False},
        # densities of fragments of different sizes in one batch
        {"name": "uneven_bf16f", "kind": "uneven", "e0": 8, "e1": 12, "e2": 16, "p": 4, "nrhs": 96, "h": 1.0,
         "precision": "bf16f_pc"},
        # FP32 V-cycle under FP64 CG on a box of unequal sides
        {"name": "box_fp32_pc", "kind": "solve", "ex": 24, "ey": 20, "ez": 28, "p": 4, "nrhs": 24, "h": 1.0,
         "precision": "fp32_pc", "guess": False, "gl": False},
        # half of the benchmark's workload: pair densities on 32^3 elements of degree 4
        {"name": "heldout32_bf16f", "kind": "solve", "ex": 32, "ey": 32, "ez": 32, "p": 4, "nrhs": 64, "h": 1.0,
         "precision": "bf16f_pc", "guess": True, "gl": False},
        # Dirichlet data of the 36 pair densities by quadrature
        {"name": "boundary36", "kind": "boundary", "ex": 16, "ey": 16, "ez": 16, "p": 4, "nrhs": 36, "h": 1.0},
        # the pair solves on the adaptive octree mesh
        {"name": "octree36_fp32_pc", "kind": "octree", "ne": 8, "q": 4, "depth": 3, "norb": 8, "precision": "fp32_pc",
         "g": True},
        # projections on a basis and the compressed exchange
        {"name": "consumers256", "kind": "consumers", "ex": 16, "ey": 16, "ez": 16, "p": 4, "nbasis": 256, "nu": 8,
         "nocc": 8, "h": 1.0},
        # one training batch of the guess network on the 16^3 mesh
        {"name": "network_16e", "kind": "network", "e": 16, "batch": 12},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _box(rng, big):
    """Elements per axis: 3..8 on the coarsest mesh, which is halved up to ``big`` times."""
    m = rng.randint(0, big)
    k = rng.randint(3, 8)
    return [2 ** m * max(3, min(8, k + rng.randint(-2, 2))) for _ in range(3)]


def draw(rng):
    kind = rng.choices(["solve", "exchange", "uneven", "boundary", "octree", "consumers", "network"],
                       [40, 10, 7, 12, 13, 9, 9])[0]
    h = round(rng.uniform(0.8, 1.25), 3)
    if kind == "solve":
        p = rng.choices([1, 2, 3, 4, 5, 6, 7], [4, 10, 10, 56, 10, 5, 5])[0]
        prec = rng.choice(["fp64", "fp32_pc", "bf16f_pc"])
        gl = rng.random() < 0.12
        E = _box(rng, 2 if p <= 4 and not gl else 1)
        cost = E[0] * E[1] * E[2] * (p + 1) ** 3 * (2.2 if prec == "fp64" else 1.3) * (1 if p in (1, 2, 4) else 3)
        most = int(2.5e8 / (cost * (6 if gl else 1)))
        return {"kind": kind, "ex": E[0], "ey": E[1], "ez": E[2], "p": p, "nrhs": _log_int(rng, 1, min(128, most)),
                "h": h, "precision": prec, "guess": False, "gl": gl}
    if kind == "exchange":
        if rng.random() < 0.5:   # the mesh of the trained guess
            E, h, guess = [16, 16, 16], 1.0, True
        else:
            E, guess = _box(rng, 1), False
        return {"kind": kind, "ex": E[0], "ey": E[1], "ez": E[2], "p": 4, "norb": rng.randint(2, 12), "h": h,
                "precision": rng.choice(["fp64", "fp32_pc", "bf16f_pc"]), "guess": guess}
    if kind == "uneven":
        e = sorted(2 * rng.randint(2, 8) for _ in range(3))
        return {"kind": kind, "e0": e[0], "e1": e[1], "e2": e[2], "p": rng.choice([3, 4, 4, 4]),
                "nrhs": _log_int(rng, 6, 128), "h": h, "precision": rng.choice(["fp64", "fp32_pc", "bf16f_pc"])}
    if kind == "boundary":
        E = _box(rng, 1)
        return {"kind": kind, "ex": E[0], "ey": E[1], "ez": E[2], "p": rng.choice([3, 4, 4, 4, 5]),
                "nrhs": _log_int(rng, 1, 64), "h": h}
    if kind == "octree":
        return {"kind": kind, "ne": rng.randint(4, 8), "q": rng.choice([2, 3, 4, 4, 4]), "depth": rng.randint(1, 3),
                "norb": rng.randint(1, 8), "precision": rng.choice(["fp64", "fp32_pc"]), "g": rng.random() < 0.7}
    if kind == "consumers":
        E = _box(rng, 1)
        return {"kind": kind, "ex": E[0], "ey": E[1], "ez": E[2], "p": rng.choice([2, 3, 4, 4]),
                "nbasis": _log_int(rng, 8, 300), "nu": rng.randint(1, 24), "nocc": rng.randint(1, 24), "h": h}
    return {"kind": kind, "e": rng.choice([8, 16, 16, 24]), "batch": rng.randint(1, 16)}


# ---- grids and densities (plain numpy / torch; shared by the inputs and the exact results)

@functools.lru_cache(maxsize=None)
def _nodes(p, gl):
    """Gauss-Lobatto (or Gauss) nodes and weights of degree p on [-1, 1]."""
    if gl:
        return np.polynomial.legendre.leggauss(p + 1)
    P = np.polynomial.legendre.Legendre.basis(p)
    x = np.concatenate([[-1.0], np.sort(P.deriv().roots().real) if p > 1 else [], [1.0]])
    return x, 2.0 / (p * (p + 1) * P(x) ** 2)


def _dims(case, k=None):
    if case["kind"] == "uneven":
        return (case["e%d" % k],) * 3
    if case["kind"] == "network":
        return (case["e"],) * 3
    return case["ex"], case["ey"], case["ez"]


def _mesh(E, p, h):
    half = [0.5 * e * h for e in E]
    return list(E), p, [-v for v in half], half


def _axes(E, h, p, gl):
    x, _ = _nodes(p, gl)
    return [torch.as_tensor(((np.arange(e)[:, None] + 0.5 * (x + 1.0)) * h - 0.5 * e * h).reshape(-1), device="cuda")
            for e in E]


def _to_elements(u, E, n):
    """[..., Z, Y, X] -> element-major fields [..., n_dofs]."""
    lead = u.shape[:-3]
    a = u.reshape(-1, E[2], n, E[1], n, E[0], n).permute(0, 1, 3, 5, 2, 4, 6)
    return a.reshape(*lead, -1).contiguous()


def _to_grid(f, E, n):
    a = f.reshape(-1, E[2], E[1], E[0], n, n, n).permute(0, 1, 4, 2, 5, 3, 6)
    return a.reshape(-1, E[2] * n, E[1] * n, E[0] * n)


def _points(E, h, p, gl):
    """Node coordinates [3, n_dofs] (field order) and boundary points [3, n_face] (face order)."""
    x, y, z = _axes(E, h, p, gl)
    n = p + 1
    Z, Y, X = torch.meshgrid(z, y, x, indexing="ij")
    xyz = _to_elements(torch.stack([X, Y, Z]), E, n)
    faces = []
    for d, other in ((0, (z, y)), (1, (z, x)), (2, (y, x))):
        A, B = (t.reshape(-1) for t in torch.meshgrid(*other, indexing="ij"))
        for side in (-0.5, 0.5):
            F = torch.full_like(A, side * E[d] * h)
            faces.append(torch.stack([F, B, A] if d == 0 else [B, F, A] if d == 1 else [B, A, F]))
    return xyz, torch.cat(faces, 1)


def _erf_over_r(c, d):
    t = c * d
    return torch.where(t < 1e-6, 2 / math.sqrt(math.pi) * c * (1 - t * t / 3), torch.erf(t) / d.clamp_min(1e-300))


def _exponents(rng, n):
    return np.exp(rng.uniform(math.log(0.3), math.log(10.0), n))


def _densities(rng, xyz, fxyz, n, reach):
    """n sums of 2..5 normalised Gaussians at the nodes, and their potentials at the boundary points."""
    rho = torch.zeros((n, xyz.shape[1]), dtype=torch.float64, device="cuda")
    g = torch.zeros((n, fxyz.shape[1]), dtype=torch.float64, device="cuda")
    for k in range(n):
        m = int(rng.integers(2, 6))
        for w, a, c in zip(rng.uniform(0.5, 1.5, m), _exponents(rng, m), rng.uniform(-1, 1, (m, 3)) * reach):
            c = torch.as_tensor(c, device="cuda")[:, None]
            rho[k] += w * (a / math.pi) ** 1.5 * torch.exp(-a * ((xyz - c) ** 2).sum(0))
            g[k] += w * _erf_over_r(math.sqrt(a), ((fxyz - c) ** 2).sum(0).sqrt())
    return rho, g


class _Orbitals:
    """Orthonormal combinations of normalised s Gaussians, three at each of some atoms."""

    def __init__(self, rng, atoms, reach, norb, centres=None, alpha=None):
        if centres is None:
            centres = np.repeat(rng.uniform(-1, 1, (atoms, 3)) * reach, 3, axis=0)
            alpha = _exponents(rng, 3 * atoms)
        self.c, self.a, self.n = centres, alpha, (2 * alpha / math.pi) ** 0.75
        s = self.a[:, None] + self.a[None]
        self.mu = self.a[:, None] * self.a[None] / s
        d2 = ((self.c[:, None] - self.c[None]) ** 2).sum(-1)
        self.pre = self.n[:, None] * self.n[None] * np.exp(-self.mu * d2)
        C = rng.standard_normal((len(alpha), norb))
        lam, U = np.linalg.eigh(C.T @ (self.pre * (math.pi / s) ** 1.5) @ C)
        self.C = C @ (U * lam ** -0.5) @ U.T
        self.norb = norb

    def values(self, xyz):
        out = torch.zeros((self.norb, xyz.shape[1]), dtype=torch.float64, device=xyz.device)
        C = torch.as_tensor(self.C, device=xyz.device)
        for k in range(len(self.a)):
            r2 = ((xyz - torch.as_tensor(self.c[k], device=xyz.device)[:, None]) ** 2).sum(0)
            out += C[k][:, None] * (self.n[k] * torch.exp(-self.a[k] * r2))
        return out

    def pairs(self):
        return [(i, j) for i in range(self.norb) for j in range(i, self.norb)]

    def potentials(self, xyz, pairs):
        """Full-space potentials of the pair densities phi_i phi_j at the points."""
        ia, ib = np.triu_indices(len(self.a))
        s = self.a[ia] + self.a[ib]
        P = (self.a[ia][:, None] * self.c[ia] + self.a[ib][:, None] * self.c[ib]) / s[:, None]
        amp = self.pre[ia, ib] * (math.pi / s) ** 1.5
        coef = np.array([self.C[ia, i] * self.C[ib, j] + (ia != ib) * self.C[ib, i] * self.C[ia, j] for i, j in pairs])
        out = torch.zeros((len(pairs), xyz.shape[1]), dtype=torch.float64, device="cuda")
        W, Pt, root = (torch.as_tensor(v, device="cuda") for v in (coef * amp, P, np.sqrt(s)))
        for t in range(0, len(s), 256):
            d = sum((xyz[k][None] - Pt[t:t + 256, k:k + 1]) ** 2 for k in range(3)).sqrt()
            out += W[:, t:t + 256] @ _erf_over_r(root[t:t + 256, None], d)
        return out


def _reach(E, h):
    return np.array([0.25 * e * h for e in E])


def _orbitals(case, rng):
    E = _dims(case)
    return _Orbitals(rng, 24 if max(E) > 20 else 8, _reach(E, case["h"]), case.get("norb", 8))


def _inputs(case, seed):
    """The inputs of a uniform-mesh case on the GPU."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "uneven":
        ids = rng.permutation(np.arange(case["nrhs"]) % 3)
        parts = []
        for k in range(3):
            xyz, fxyz = _points(_dims(case, k), case["h"], case["p"], False)
            parts.append([iter(v) for v in _densities(rng, xyz, fxyz, int((ids == k).sum()),
                                                      _reach(_dims(case, k), case["h"]))])
        rho, g = zip(*((next(parts[k][0]), next(parts[k][1])) for k in ids))
        return {"ids": [int(k) for k in ids], "rho": torch.cat(rho), "g": torch.cat(g)}
    E = _dims(case)
    xyz, fxyz = _points(E, case["h"], case["p"], bool(case.get("gl")))
    if kind == "exchange":
        orb = _orbitals(case, rng)
        return {"phi": orb.values(xyz).reshape(-1), "g": orb.potentials(fxyz, orb.pairs()).reshape(-1)}
    if kind == "solve" and not (case["guess"] and case["nrhs"] > 8):
        rho, g = _densities(rng, xyz, fxyz, case["nrhs"], _reach(E, case["h"]))
        return {"rho": rho.reshape(-1), "g": g.reshape(-1)}
    if kind in ("solve", "boundary"):
        # pair densities of as many molecules as the batch needs
        rho, g, left = [], [], case["nrhs"]
        while left > 0:
            orb = _orbitals(case, rng)
            pairs = orb.pairs()[:left]
            phi = orb.values(xyz)
            rho += [phi[i] * phi[j] for i, j in pairs]
            if kind == "solve":
                g.append(orb.potentials(fxyz, pairs))
            left -= len(pairs)
        return {"rho": torch.cat(rho), "g": torch.cat(g).reshape(-1) if g else None}
    # consumers: basis fields, vectors, occupied orbitals, a Hartree potential and W = V psi for a
    # positive potential V (so that the compressed exchange is positive definite)
    gen = torch.Generator("cuda").manual_seed(int(seed) % (1 << 31))
    nd = xyz.shape[1]
    r = (xyz ** 2).sum(0).sqrt()
    smooth = torch.exp(-0.1 * r * r)
    phi = torch.randn((case["nbasis"], nd), dtype=torch.float64, device="cuda", generator=gen) * smooth
    u = torch.randn((case["nu"], nd), dtype=torch.float64, device="cuda", generator=gen) * smooth
    psi = _Orbitals(rng, 8, _reach(E, case["h"]), case["nocc"]).values(xyz)
    V = _erf_over_r(1.0, r) + 0.1
    return {"phi": phi.reshape(-1), "u": u.reshape(-1), "psi": psi.reshape(-1), "vH": V, "W": (V * psi).reshape(-1)}


# ---- the octree case: the mesh follows a fixed molecule, the right-hand sides the seed's orbitals

def _octree_molecule(case):
    rng = np.random.default_rng(2)
    reach = 0.5 * case["ne"]
    return np.repeat(rng.uniform(-reach, reach, (8, 3)), 3, axis=0), _exponents(rng, 24)


def _octree(case):
    centres, alpha = _octree_molecule(case)
    orb = _Orbitals(np.random.default_rng(3), 8, 0.0, 8, centres, alpha)

    def density(x, y, z):
        v = orb.values(torch.as_tensor(np.stack([x, y, z]), device="cuda"))
        return (v * v).sum(0).cpu().numpy()

    ne = case["ne"]
    return binding.Octree((ne,) * 3, (-float(ne),) * 3, (float(ne),) * 3, q=case["q"], rho=density, delta_q=1e-8,
                          max_depth=case["depth"], precision=case["precision"], rtol=RTOL, cheb_degree=8,
                          cheb_degree_h=4)


@functools.lru_cache(maxsize=None)
def _octree_size(ne, q, depth):
    o = _octree({"ne": ne, "q": q, "depth": depth, "precision": "fp64"})
    size = o.n_dofs, o.n_boundary
    o.close()
    return size


# ---- the guess network

def _layers(levels=4, c=32, cin=125, cout=27):
    """(kernel, stride, inputs, outputs) of every convolution in parameter order."""
    out = [(1, 1, cin, c)]
    for k in range(levels):
        out += [(3, 1, c, c)] * 2 + ([(3, 2, c, c)] if k < levels - 1 else [])
    for _ in range(levels - 1):
        out += [(3, 1, c, c), (3, 1, 2 * c, c)]
    return out + [(1, 1, c, cout)]


def _network_inputs(case, seed):
    rng = np.random.default_rng(seed)
    params = np.concatenate([v for k, s, ci, co in _layers() for v in (
        math.sqrt(2.0 / (k ** 3 * ci)) * rng.standard_normal(k ** 3 * ci * co), 0.02 * rng.standard_normal(co))])
    E = (case["e"],) * 3
    # densities at the degree-4 nodes, and at the output's degree-2 nodes the gradient of the squared
    # error of a prediction that is still small: minus the potential
    rho, v = _densities(rng, _points(E, 1.0, 4, False)[0], _points(E, 1.0, 2, False)[0], case["batch"], _reach(E, 1.0))
    s = rho.square().mean(1, keepdim=True).sqrt()
    return {"params": params.astype(np.float32), "x": (rho / s).float().reshape(-1),
            "dy": (-v / s / v.shape[1]).float().reshape(-1)}


# ---- the interface: prepare, run, work, exact

def prepare(case, seed):
    kind = case["kind"]
    if kind == "network":
        s = _network_inputs(case, seed)
        net = binding.Net()
        net.set_params(s["params"])
        return {"case": case, "net": net, **s}
    if kind == "octree":
        o = _octree(case)
        centres, alpha = _octree_molecule(case)
        orb = _Orbitals(np.random.default_rng(seed), 8, 0.0, case["norb"], centres, alpha)
        phi = orb.values(torch.as_tensor(o.nodes(), device="cuda"))
        f = torch.stack([phi[i] * phi[j] for i, j in orb.pairs()])
        g = orb.potentials(torch.as_tensor(o.boundary_points().copy(), device="cuda"), orb.pairs()) if case["g"] else None
        return {"case": case, "octree": o, "f": f, "g": g}
    s = _inputs(case, seed)
    meshes = [_mesh(_dims(case, k), case["p"], case["h"]) for k in range(3 if kind == "uneven" else 1)]
    opts = {"rtol": RTOL, "precision": case.get("precision", "fp64")}
    if case.get("gl"):
        opts["node_family"] = "gl"
    s["case"], s["ctx"] = case, binding.Context(meshes, **opts)
    if case.get("guess"):
        s["net"] = binding.Net()
        s["net"].load(os.path.join(WEIGHTS, "guess_%de_p4.bin" % case["ex"]))
        s["ctx"].attach_guess(s["net"])
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "solve":
        return {"v": s["ctx"].solve_batch(s["rho"], s["g"])[0]}
    if kind == "uneven":
        return {"v": s["ctx"].solve_batch(s["rho"], s["g"], mesh_ids=s["ids"])[0]}
    if kind == "exchange":
        W, K, ex, _, _ = s["ctx"].exchange(s["phi"], s["g"])
        return {"W": W, "K": K, "E_x": ex}
    if kind == "boundary":
        return {"g": s["ctx"].boundary_data(s["rho"])}
    if kind == "octree":
        return {"v": s["octree"].solve(s["octree"].rhs(s["f"], s["g"]))[0]}
    if kind == "consumers":
        ctx = s["ctx"]
        hartree = ctx.hartree_action(s["phi"], s["u"], s["vH"])
        xi = ctx.ace_build(s["psi"], s["W"])
        return {"hartree": hartree, "xi": xi, "ace": ctx.ace_action(s["phi"], s["u"], xi)}
    y = s["net"].forward(s["x"], _dims(case), case["batch"])
    return {"y": y, "grad": s["net"].backward(s["dy"])}


def work(case):
    """Inputs and outputs once, and the operations of the method: for solves, 13 iterations of 13
    finest-level operator applications at 6 (p + 1) operations per node."""
    kind = case["kind"]
    if kind == "network":
        vox, flops, scale = case["e"] ** 3 * case["batch"], 0, 1.0
        for k, s, ci, co in _layers():
            scale = scale / 8 if s == 2 else scale
            flops += 2 * k ** 3 * ci * co * vox * scale
        return {"bytes": 4 * vox * (125 + 27 + 27) + 8 * sum(k ** 3 * ci * co + co for k, _, ci, co in _layers()),
                "flops": 3 * flops}
    if kind == "octree":
        nd, nb = _octree_size(case["ne"], case["q"], case["depth"])
        n = case["norb"] * (case["norb"] + 1) // 2
        return {"bytes": 8 * n * (2 * nd + nb), "flops": 169 * 6 * (case["q"] + 1) * nd * n}
    p = case["p"]

    def sizes(E):
        nx, ny, nz = (e * (p + 1) for e in E)
        return nx * ny * nz, 2 * (nx * ny + ny * nz + nx * nz)

    if kind == "uneven":
        per = [sizes(_dims(case, k)) for k in range(3)]
        count = [len(range(k, case["nrhs"], 3)) for k in range(3)]
        return {"bytes": 8 * sum(c * (2 * nd + nf) for c, (nd, nf) in zip(count, per)),
                "flops": sum(169 * 6 * (p + 1) * nd * c for c, (nd, nf) in zip(count, per))}
    nd, nf = sizes(_dims(case))
    if kind == "solve":
        return {"bytes": 8 * case["nrhs"] * (2 * nd + nf), "flops": 169 * 6 * (p + 1) * nd * case["nrhs"]}
    if kind == "exchange":
        n, pairs = case["norb"], case["norb"] * (case["norb"] + 1) // 2
        return {"bytes": 8 * (2 * n * nd + pairs * nf), "flops": 169 * 6 * (p + 1) * nd * pairs + 4 * n * n * nd}
    if kind == "boundary":
        return {"bytes": 8 * case["nrhs"] * (nd + nf), "flops": float(nd) * nf * (9 + 2 * case["nrhs"])}
    nb, nu, no = case["nbasis"], case["nu"], case["nocc"]
    return {"bytes": 8 * nd * (nb + nu + 3 * no + 1), "flops": 2 * nd * (nb * (nu + no) + no * (nu + 2 * no))}


def _axis_matrix(e, h, p, gl):
    """1D interior-penalty matrix, masses and boundary lifts of e elements of width h."""
    x, w = _nodes(p, gl)
    n, J, sg = p + 1, 0.5 * h, 8.0 * (p + 1) ** 2 / h
    polys = [np.polynomial.Polynomial.fromroots(np.delete(x, j)) for j in range(n)]
    polys = [q / q(x[j]) for j, q in enumerate(polys)]
    D = np.array([[q.deriv()(t) / J for q in polys] for t in x])
    ends = {s: (np.array([q(t) for q in polys]), np.array([q.deriv()(t) / J for q in polys]))
            for s, t in ((0, -1.0), (1, 1.0))}
    A = np.kron(np.eye(e), D.T @ (J * w[:, None] * D))

    def spread(k, s):
        jump, slope = np.zeros(e * n), np.zeros(e * n)
        jump[k * n:k * n + n], slope[k * n:k * n + n] = ends[s]
        return jump, slope

    lifts = []
    for k in range(e + 1):   # the face left of element k
        if 0 < k < e:
            (ul, sl), (ur, sr) = spread(k - 1, 1), spread(k, 0)
            jump, slope = ul - ur, 0.5 * (sl + sr)
        else:
            u, s = spread(0, 0) if k == 0 else spread(e - 1, 1)
            jump, slope = u, (-s if k == 0 else s)   # outward derivative
            lifts.append(sg * jump - slope)
        A += sg * np.outer(jump, jump) - np.outer(jump, slope) - np.outer(slope, jump)
    return A, np.tile(J * w, e), lifts


def _exact_solve(E, h, p, gl, rho, g):
    """A^-1 b of the discrete problems by diagonalising the three 1D pencils; fields in and out."""
    n = p + 1
    ax = [_axis_matrix(e, h, p, gl) for e in E]
    dev = [[torch.as_tensor(v, device="cuda") for v in (A, m, l0, l1)] for A, m, (l0, l1) in ax]
    (_, mx, *lx), (_, my, *ly), (_, mz, *lz) = dev
    Q, lam = [], []
    for A, m, _ in ax:
        r = m ** -0.5
        val, vec = np.linalg.eigh(r[:, None] * A * r[None])
        Q.append(torch.as_tensor(r[:, None] * vec, device="cuda"))
        lam.append(torch.as_tensor(val, device="cuda"))
    denom = lam[2][:, None, None] + lam[1][None, :, None] + lam[0][None, None]
    N = [e * n for e in E]
    faces = [(N[2], N[1])] * 2 + [(N[2], N[0])] * 2 + [(N[1], N[0])] * 2
    out = torch.empty_like(rho)
    M = mz[:, None, None] * my[None, :, None] * mx[None, None]
    for k in range(rho.shape[0]):
        b = 4 * math.pi * M * _to_grid(rho[k], E, n)[0]
        F = [t.reshape(s) for t, s in zip(torch.split(g[k], [a * c for a, c in faces]), faces)]
        for side in (0, 1):
            b += lx[side][None, None] * (mz[:, None] * my[None] * F[side])[:, :, None]
            b += ly[side][None, :, None] * (mz[:, None] * mx[None] * F[2 + side])[:, None]
            b += lz[side][:, None, None] * (my[:, None] * mx[None] * F[4 + side])[None]
        t = torch.matmul(Q[1].T.contiguous(), b @ Q[0])
        t = (Q[2].T.contiguous() @ t.reshape(N[2], -1)).reshape(N[2], N[1], N[0]) / denom
        t = torch.matmul(Q[1], t @ Q[0].T.contiguous())
        out[k] = _to_elements((Q[2] @ t.reshape(N[2], -1)).reshape(N[2], N[1], N[0]), E, n)
    return out


def _weights(E, h, p):
    w = torch.as_tensor(0.5 * h * _nodes(p, False)[1], device="cuda")
    one = (w[:, None, None] * w[None, :, None] * w[None, None]).reshape(-1)
    return one.repeat(E[0] * E[1] * E[2])


def _exact_network(case, s):
    """The network in 64 bits: convolutions as sums over the taps."""
    c, e, at = 32, case["e"], 0
    P = torch.as_tensor(s["params"], device="cuda").double().requires_grad_()
    todo = iter(_layers())

    def conv(u, relu=True):
        nonlocal at
        k, st, ci, co = next(todo)
        W, at = P[at:at + k ** 3 * ci * co].reshape(k, k, k, ci, co), at + k ** 3 * ci * co
        bias, at = P[at:at + co], at + co
        if k == 1:
            y = u @ W[0, 0, 0] + bias
        else:
            m = [v // st for v in u.shape[1:4]]
            up = torch.nn.functional.pad(u, (0, 0, 1, 1, 1, 1, 1, 1))
            y = bias
            for a in range(3):
                for b in range(3):
                    for d in range(3):
                        y = y + up[:, a:a + st * m[0]:st, b:b + st * m[1]:st, d:d + st * m[2]:st] @ W[a, b, d]
        return torch.relu(y) if relu else y

    hcur, skip = conv(s["x"].double().reshape(case["batch"], e, e, e, 125)), []
    for k in range(4):
        skip.append(conv(conv(hcur)))
        hcur = conv(skip[-1]) if k < 3 else None
    d = skip[3]
    for k in (2, 1, 0):
        up = d.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)
        d = conv(torch.cat([conv(up), skip[k]], -1))
    y = conv(d, relu=False).reshape(-1)
    y.backward(s["dy"].double())
    return {"y": y.detach(), "grad": P.grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "octree":
        return None   # its matrix (hanging faces integrated piece by piece) has no short plain form
    if kind == "network":
        return _exact_network(case, _network_inputs(case, seed))
    s, p, h = _inputs(case, seed), case["p"], case["h"]
    if kind == "uneven":
        nd = [(e * (p + 1)) ** 3 for e in (case["e0"], case["e1"], case["e2"])]
        nf = [6 * (e * (p + 1)) ** 2 for e in (case["e0"], case["e1"], case["e2"])]
        rho, g = torch.split(s["rho"], [nd[k] for k in s["ids"]]), torch.split(s["g"], [nf[k] for k in s["ids"]])
        return {"v": torch.cat([_exact_solve(_dims(case, k), h, p, False, r[None], f[None])[0]
                                for k, r, f in zip(s["ids"], rho, g)])}
    E = _dims(case)
    nd = E[0] * E[1] * E[2] * (p + 1) ** 3
    if kind == "solve":
        rho, g = s["rho"].reshape(-1, nd), s["g"].reshape(case["nrhs"], -1)
        return {"v": _exact_solve(E, h, p, bool(case["gl"]), rho, g).reshape(-1)}
    w = _weights(E, h, p)
    if kind == "exchange":
        n = case["norb"]
        phi = s["phi"].reshape(n, nd)
        pairs = [(i, j) for i in range(n) for j in range(i, n)]
        v = _exact_solve(E, h, p, False, torch.stack([phi[i] * phi[j] for i, j in pairs]),
                         s["g"].reshape(len(pairs), -1))
        W, K = torch.zeros_like(phi), []
        for q, (i, j) in enumerate(pairs):
            W[i] += phi[j] * v[q]
            if i != j:
                W[j] += phi[i] * v[q]
            K.append((w * phi[i] * phi[j] * v[q]).sum())
        K = torch.stack(K)
        twice = torch.tensor([1.0 if i == j else 2.0 for i, j in pairs], dtype=torch.float64, device="cuda")
        return {"W": W.reshape(-1), "K": K, "E_x": float((K * twice).sum())}
    if kind == "boundary":
        # the term of a node at the boundary point itself is left out
        xyz, fxyz = _points(E, h, p, False)
        f = (s["rho"].reshape(-1, nd) * w).T.contiguous()
        g = torch.empty((fxyz.shape[1], f.shape[1]), dtype=torch.float64, device="cuda")
        step = max(16, int(1.5e8 // nd))
        for t in range(0, fxyz.shape[1], step):
            d = sum((fxyz[k, t:t + step, None] - xyz[k][None]) ** 2 for k in range(3)).sqrt()
            g[t:t + step] = torch.where(d < 1e-6 * h, 0.0, 1.0 / d) @ f
        return {"g": g.T.contiguous().reshape(-1)}
    phi, u, psi, W = (s[k].reshape(-1, nd) for k in ("phi", "u", "psi", "W"))
    M = (w * psi) @ W.T
    xi = torch.linalg.solve_triangular(torch.linalg.cholesky(0.5 * (M + M.T)), W, upper=False)
    return {"hartree": (w * s["vH"] * phi) @ u.T, "xi": xi.reshape(-1), "ace": ((w * phi) @ xi.T) @ ((w * xi) @ u.T)}
