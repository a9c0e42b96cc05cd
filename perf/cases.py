"""The workloads this library's performance is measured on, and plain FP64
references of their results.

Each case is one pass through the package's public entry points, from the
smallest call (one spinor on 4^4, where launches count) to a whole noise
vector of the 16^3x32 lattice.  Lattice extents are even (the library's
rule); the ragged ones leave a partial wave of sites and a partial workgroup
of right-hand sides.  Gauge fields are SU(3) links exp(i eps H) with Gaussian
H, drawn from the seed on the GPU; kappa stays below the critical value of
each eps, so every seed's solves converge in a similar number of iterations.
"""
import math

import numpy as np
import torch

import paper_1108_2473_amd as fl

DEV = "cuda:0"
PREC = {"f64": fl.PREC_F64, "f32": fl.PREC_F32, "h16": fl.PREC_H16}
SOLVER = {"bicgstab": fl.SOLVER_BICGSTAB, "cgnr": fl.SOLVER_CGNR}
DILUTION = {"none": 0, "spin-colour": fl.DIL_SPIN | fl.DIL_COLOUR,
            "time-spin-colour": fl.DIL_TIME | fl.DIL_SPIN | fl.DIL_COLOUR, "even-odd": fl.DIL_EVENODD,
            "cubic": fl.DIL_CUBIC}
NOISE = {"z4": fl.NOISE_Z4, "cz2": fl.NOISE_CZ2, "z2": fl.NOISE_Z2}
G6 = list(fl.GAMMAS_PAPER)
# the 33 momenta of the disconnected two-point function: all n with entries
# -1, 0, 1 and the six (+-2, 0, 0) ones
MOM = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]
MOM += [(2, 0, 0), (0, 2, 0), (0, 0, 2), (-2, 0, 0), (0, -2, 0), (0, 0, -2)]


def listed():
    return [
        # one Wilson-Dirac operator on the smallest lattice of the tests: what a call costs by itself
        dict(name="apply_4x4x4x4_1", kind="apply", lattice="4x4x4x4", eps=0.5, kappa=0.12, nrhs=1, dagger=False),
        # the operator on a whole propagator (12 spin-colour columns) of the paper's lattice
        dict(name="apply_16x16x16x32_12", kind="apply", lattice="16x16x16x32", eps=0.6, kappa=0.157, nrhs=12,
             dagger=True),
        # one reference solve in FP64 throughout
        dict(name="solve_f64_8x8x8x16_1", kind="solve", lattice="8x8x8x16", eps=0.5, kappa=0.14, nrhs=1, prec="f64",
             solver="bicgstab"),
        # a propagator at the paper's kappa with the library's default solver
        dict(name="solve_f32_16x16x16x32_12", kind="solve", lattice="16x16x16x32", eps=0.6, kappa=0.157, nrhs=12,
             prec="f32", solver="bicgstab"),
        # a ragged lattice and batch with the benchmark's solver
        dict(name="solve_h16_10x6x14x18_7", kind="solve", lattice="10x6x14x18", eps=0.5, kappa=0.14, nrhs=7,
             prec="h16", solver="cgnr"),
        # exact loops of one whole timeslice: 6144 point sources
        dict(name="exact_8x8x8x16", kind="exact", lattice="8x8x8x16", eps=0.5, kappa=0.14, slices=1, batch=768,
             prec="h16", solver="cgnr"),
        # the benchmark's step at the paper's kappa, for 16 of its 32 timeslices (192 diluted sources)
        dict(name="stochastic_16x16x16x32", kind="stochastic", lattice="16x16x16x32", eps=0.6, kappa=0.157,
             noise="z4", dilution="time-spin-colour", nlp=1, tb=0, te=16, prec="h16", solver="cgnr"),
        # the truncated solver method on three uneven lattices in one launch sequence
        dict(name="tsm_uneven", kind="tsm", lattice="8x8x8x8+12x12x12x24+16x16x16x32", eps=0.6, kappa=0.14,
             noise="cz2", dilution="none", nlp=64, nhp=4),
        # training the links on exact loops: gradient of a few sites' loops (12 solves each)
        dict(name="grad_12x12x12x24", kind="grad", lattice="12x12x12x24", eps=0.5, kappa=0.14, sites=32, batch=768,
             prec="h16", solver="cgnr"),
        # Gaussian smearing of a propagator with the paper's alpha and n
        dict(name="smear_16x16x16x32_12", kind="smear", lattice="16x16x16x32", eps=0.6, nrhs=12, alpha=4.0, n=50),
        # the connected correlator: APE-smeared links, smeared source, 12 solves, smeared sink, projection
        dict(name="pion_16x16x16x32", kind="pion", lattice="16x16x16x32", eps=0.6, kappa=0.157, alpha=4.0, n=50,
             ape=20, prec="h16", solver="cgnr"),
        # the disconnected correlator of two loop sets
        dict(name="corr_16x16x16x32", kind="corr", lattice="16x16x16x32", ngamma=6, nmom=33),
    ]


def _even(rng, lo, hi):
    return 2 * max(lo // 2, min(hi // 2, round(0.5 * math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _lattice(rng, xlo, xhi, tlo, thi):
    return "x".join(str(_even(rng, lo, hi)) for lo, hi in ((xlo, xhi),) * 3 + ((tlo, thi),))


def _log(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["apply", "apply", "solve", "solve", "exact", "stochastic", "tsm", "grad", "smear", "pion", "corr"])
    eps = rng.choice([0.5, 0.55, 0.6])
    c = dict(kind=kind, eps=eps)
    prec, solver = rng.choice([("f64", "bicgstab"), ("f32", "bicgstab"), ("f32", "cgnr"), ("h16", "cgnr"),
                               ("f64", "cgnr")])
    kappa = rng.choice([0.12, 0.13, 0.135])
    if kind == "apply":
        c.update(lattice=_lattice(rng, 4, 16, 4, 32), kappa=kappa, nrhs=_log(rng, 1, 48), dagger=rng.random() < 0.5)
    elif kind == "solve":
        c.update(lattice=_lattice(rng, 4, 16, 4, 32), kappa=kappa, nrhs=_log(rng, 1, 24), prec=prec, solver=solver)
    elif kind == "exact":
        c.update(lattice=_lattice(rng, 4, 8, 4, 16), kappa=kappa, slices=rng.choice([1, 2]),
                 batch=rng.choice([192, 384, 768]), prec=prec if prec != "f64" else "f32", solver=solver)
        if c["slices"] * _vol(_dims(c["lattice"])[:3]) > 512:
            c["slices"] = 1
    elif kind == "stochastic":
        lat = _lattice(rng, 6, 16, 6, 32)
        dil, noise = rng.choice(["spin-colour", "time-spin-colour", "even-odd", "cubic"]), rng.choice(["z4", "cz2", "z2"])
        tb = rng.randrange(0, 3)
        c.update(lattice=lat, kappa=kappa, noise=noise, dilution=dil, nlp=_log(rng, 1, 6), tb=tb,
                 te=rng.randrange(tb + 1, _dims(lat)[3] + 1), prec="h16" if solver == "cgnr" else "f32", solver=solver)
        if dil == "time-spin-colour":
            c["nlp"] = 1
    elif kind == "tsm":
        c.update(lattice="+".join(_lattice(rng, 6, 14, 6, 28) for _ in range(rng.choice([1, 2, 3]))), kappa=kappa,
                 noise=rng.choice(["z4", "cz2", "z2"]), dilution=rng.choice(["none", "even-odd"]),
                 nlp=_log(rng, 4, 48), nhp=_log(rng, 1, 6))
    elif kind == "grad":
        c.update(lattice=_lattice(rng, 4, 12, 4, 20), kappa=kappa, sites=_log(rng, 1, 24),
                 batch=rng.choice([192, 384, 768]), prec=prec, solver=solver)
    elif kind == "smear":
        c.update(lattice=_lattice(rng, 4, 16, 4, 32), nrhs=_log(rng, 1, 24), alpha=rng.choice([2.0, 4.0]),
                 n=_log(rng, 5, 50))
    elif kind == "pion":
        c.update(lattice=_lattice(rng, 6, 14, 8, 28), kappa=kappa, alpha=rng.choice([2.0, 4.0]), n=_log(rng, 5, 50),
                 ape=_log(rng, 2, 20), prec=prec if prec != "f64" else "f32", solver=solver)
    else:
        c.update(lattice=_lattice(rng, 4, 24, 4, 48), ngamma=rng.choice([1, 2, 6, 16]), nmom=_log(rng, 1, 33))
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dims(text):
    return tuple(int(v) for v in text.split("x"))


def _vol(dims):
    return int(np.prod(dims))


def _gen(seed, stream=0):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + stream)


def _randn(shape, g):
    return torch.randn(tuple(shape) + (2,), dtype=torch.float64, device=DEV, generator=g).mul_(math.sqrt(0.5))


def _complex(shape, g):
    return torch.view_as_complex(_randn(shape, g))


def _mm(a, b):
    """Products of 3x3 matrices over leading axes."""
    return sum(a[..., :, k, None] * b[..., k, None, :] for k in range(3))


def _links(dims, eps, g):
    """exp(i eps H), H Hermitian traceless with Gaussian coefficients of the
    eight generators, re-unitarised: [4][V][3][3]."""
    V = _vol(dims)
    h = torch.randn((4, V, 8), dtype=torch.float64, device=DEV, generator=g)
    H = torch.zeros((4, V, 3, 3), dtype=torch.complex128, device=DEV)
    for a, (i, j) in ((0, (0, 1)), (3, (0, 2)), (5, (1, 2))):
        z = torch.complex(h[..., a], -h[..., a + 1]) * 0.5
        H[..., i, j] = z
        H[..., j, i] = z.conj()
    H[..., 0, 0] = (h[..., 2] + h[..., 7] / math.sqrt(3)) * 0.5
    H[..., 1, 1] = (-h[..., 2] + h[..., 7] / math.sqrt(3)) * 0.5
    H[..., 2, 2] = -h[..., 7] / math.sqrt(3)
    A = H * (1j * eps / 16)
    U = torch.eye(3, dtype=torch.complex128, device=DEV).expand(H.shape).clone()
    T = U
    for k in range(1, 13):
        T = _mm(T, A) / k
        U = U + T
    for _ in range(4):
        U = _mm(U, U)
    r0 = U[..., 0, :]
    r0 = r0 / r0.abs().square().sum(-1, keepdim=True).sqrt()
    r1 = U[..., 1, :]
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=-2).contiguous()


def _point_columns(dims, nrhs, g):
    """Right-hand sides as a propagator has them: unit point sources, one
    spin-colour column each, 12 per site."""
    b = torch.zeros((nrhs, _vol(dims), 4, 3), dtype=torch.complex128, device=DEV)
    s = torch.randint(0, _vol(dims), ((nrhs + 11) // 12,), device=DEV, generator=g).tolist()
    for k in range(nrhs):
        b[k, s[k // 12], (k % 12) // 3, k % 3] = 1.0
    return b


def _params(case, tol=1e-12):
    p = case["prec"]
    return fl.SolverParams(tol=tol, inner_prec=PREC[p], gauge_reals=18 if p == "f64" else 12,
                           solver=SOLVER[case["solver"]], batch=case.get("batch", 0))


def _grad_weights(case, dims, g):
    """Weights of the loops of one timeslice, nonzero on `sites` sites."""
    Vs = _vol(dims[:3])
    at = torch.randperm(Vs, device=DEV, generator=g)[: min(case["sites"], Vs)]
    w = torch.zeros((2, 1, Vs), dtype=torch.complex128, device=DEV)
    w[:, 0, at] = _complex((2, at.numel()), g)
    return w


def _inputs(case, seed):
    """The arrays of a case, from the seed alone."""
    d = [_dims(t) for t in case["lattice"].split("+")]
    g = _gen(seed)
    x = dict(dims=d)
    if case["kind"] != "corr":
        x["U"] = [_links(q, case["eps"], g) for q in d]
    V = _vol(d[0])
    kind = case["kind"]
    if kind in ("apply", "smear"):
        x["psi"] = _complex((case["nrhs"], V, 4, 3), g)
    elif kind == "solve":
        x["psi"] = _point_columns(d[0], case["nrhs"], g)
    elif kind == "grad":
        x["w"] = _grad_weights(case, d[0], g)
    elif kind == "corr":
        shape = (case["ngamma"], d[0][3], _vol(d[0][:3]))
        x["L1"], x["L2"] = _complex(shape, g), _complex(shape, g)
    elif kind == "pion":
        x["y0"] = int(torch.randint(0, V, (1,), device=DEV, generator=g))
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    x["case"] = case
    x["seed"] = int(seed)
    x["lat"] = []
    for k, d in enumerate(x["dims"]):
        lat = fl.Lattice(d, -1, device=0)
        if "U" in x:
            lat.set_gauge(x["U"][k])
        if "kappa" in case:
            lat.set_kappa(case["kappa"])
        x["lat"].append(lat)
    x.pop("U", None)
    return x


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case, lat, dims = s["case"], s["lat"][0], s["dims"][0]
    kind = case["kind"]
    if kind == "apply":
        return lat.apply_D(s["psi"], dagger=case["dagger"])
    if kind == "solve":
        return lat.solve(s["psi"], _params(case))[0]
    if kind == "exact":
        return lat.loops_exact(list(range(case["slices"])), G6, _params(case))
    if kind == "stochastic":
        q = fl.NoiseParams(noise=NOISE[case["noise"]], seed=s["seed"], n_lp=case["nlp"],
                           dilution=DILUTION[case["dilution"]], t_begin=case["tb"], t_end=case["te"])
        return lat.loops_stochastic(q, G6, lp=_params(case))
    if kind == "tsm":
        qs = [fl.NoiseParams(noise=NOISE[case["noise"]], seed=s["seed"] + k, n_lp=case["nlp"], n_hp=case["nhp"],
                             dilution=DILUTION[case["dilution"]], t_begin=0, t_end=d[3])
              for k, d in enumerate(s["dims"])]
        return fl.loops_stochastic_multi(s["lat"], qs, G6, fl.SolverParams(tol=1e-3, truncated=True),
                                         fl.SolverParams(tol=1e-12))
    if kind == "grad":
        return lat.loops_grad([0], [0, 15], s["w"], _params(case))
    if kind == "smear":
        return lat.smear(s["psi"].clone(), case["alpha"], case["n"], 1.0 + 6.0 * case["alpha"])
    if kind == "pion":
        lat.ape_smear(0.5, case["ape"], want_links=False)
        return lat.pion_corr(s["y0"], _params(case), case["alpha"], case["n"], 1.0 + 6.0 * case["alpha"], True, True,
                             MOM[:7])
    mom = MOM[: case["nmom"]]
    p1 = lat.momentum_project(s["L1"], mom)
    p2 = lat.momentum_project(s["L2"], [(-a, -b, -c) for a, b, c in mom])
    return p1, p2, lat.disconnected_corr(p1, p2, [(k, k) for k in range(case["ngamma"])])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
HOP = 1320  # flop of one hopping term per output site and right-hand side
SITE = {"f64": 192, "f32": 96, "h16": 52}  # bytes of a spinor site in each iteration storage
LINK = {"f64": 144, "f32": 48, "h16": 24}


def _solve_work(V, n, prec, kappa):
    """n solves on V sites: source in, solution out, and the operator of a
    nominal number of iterations, its input and output once and every link
    once for each of its applications."""
    its = 160 if kappa > 0.15 else 50
    ops = 2 * its  # two applications of the even-odd operator an iteration
    return (2 * 192.0 * V * n + ops * (SITE[prec] * V * n + 4 * LINK[prec] * V), float(ops) * V * n * HOP)


def work(case):
    d = [_dims(t) for t in case["lattice"].split("+")]
    V = _vol(d[0])
    Vs = _vol(d[0][:3])
    kind = case["kind"]
    links = 4 * 144.0 * V
    if kind == "apply":
        by, fp = 2 * 192.0 * V * case["nrhs"] + links, float(HOP + 48) * V * case["nrhs"]
    elif kind == "solve":
        by, fp = _solve_work(V, case["nrhs"], case["prec"], case["kappa"])
    elif kind == "exact":
        n = 12 * Vs * case["slices"]
        by, fp = _solve_work(V, n, case["prec"], case["kappa"])
    elif kind == "stochastic":
        per = {"spin-colour": 12, "time-spin-colour": 12 * (case["te"] - case["tb"]), "even-odd": 2, "cubic": 8}
        by, fp = _solve_work(V, per[case["dilution"]] * case["nlp"], case["prec"], case["kappa"])
    elif kind == "tsm":
        per = 2 if case["dilution"] == "even-odd" else 1
        by = fp = 0.0
        for q in d:
            b0, f0 = _solve_work(_vol(q), per * case["nhp"], "f32", case["kappa"])
            b1, f1 = _solve_work(_vol(q), per * (case["nlp"] + case["nhp"]), "f32", case["kappa"])
            by, fp = by + b0 + 0.25 * b1, fp + f0 + 0.25 * f1  # a quarter of the iterations to 1e-3
    elif kind == "grad":
        n = 12 * min(case["sites"], Vs)
        by, fp = _solve_work(V, n, case["prec"], case["kappa"])
        by, fp = by + 2 * 192.0 * V * n + links, fp + 4 * 2 * 288.0 * V * n  # outer products of every link
    elif kind == "smear":
        by, fp = 2 * 192.0 * V * case["nrhs"] + 0.75 * links, 6 * 4 * 66.0 * V * case["nrhs"] * case["n"]
    elif kind == "pion":
        by, fp = _solve_work(V, 12, case["prec"], case["kappa"])
        by += 0.75 * 2 * links + 4 * 192.0 * V * 12
        fp += 2 * 6 * 4 * 66.0 * V * 12 * case["n"] + 3 * 4 * 2 * 2 * 198.0 * V * case["ape"]
    else:
        n = case["ngamma"] * d[0][3]
        by, fp = 2 * 16.0 * n * (Vs + case["nmom"]), 2 * 8.0 * n * Vs * case["nmom"]
    return {"bytes": by, "flops": fp}


# ---------------------------------------------------------------------------
# FP64 references, written on whole torch arrays
# ---------------------------------------------------------------------------
# rows of g_mu in the chiral basis: (column, value) of the one nonzero entry
_GAMMA = [((3, -1j), (2, -1j), (1, 1j), (0, 1j)), ((3, -1), (2, 1), (1, 1), (0, -1)),
          ((2, -1j), (3, 1j), (0, 1j), (1, -1j)), ((2, 1), (3, 1), (0, 1), (1, 1))]


def _grid(a, dims, lead):
    return a.reshape(a.shape[:lead] + dims[::-1] + a.shape[lead + 1:])


def _umul(U, psi, adj):
    """U psi (adj: U^+ psi) for links [T][Z][Y][X][3][3] and spinors [n][T][Z][Y][X][4][3]."""
    if adj:
        return sum(U[..., b, :].conj().unsqueeze(-2) * psi[..., b:b + 1] for b in range(3))
    return sum(U[..., :, b].unsqueeze(-2) * psi[..., b:b + 1] for b in range(3))


def _gmul(mu, psi):
    c = torch.tensor([v for _, v in _GAMMA[mu]], dtype=torch.complex128, device=psi.device)
    return psi[..., [k for k, _ in _GAMMA[mu]], :] * c[:, None]


def _dirac(U, psi, kappa, bc, dagger):
    s = 1 if dagger else -1
    out = psi.clone()
    for mu in range(4):
        ax = 4 - mu
        f = torch.roll(psi, -1, ax)
        if mu == 3 and bc < 0:
            f[:, -1] *= -1
        f = _umul(U[mu], f, False)
        out -= kappa * (f + s * _gmul(mu, f))
        f = torch.roll(_umul(U[mu], psi, True), 1, ax)
        if mu == 3 and bc < 0:
            f[:, 0] *= -1
        out -= kappa * (f - s * _gmul(mu, f))
    return out


def _norm2(f):
    return f.abs().square().sum(dim=tuple(range(1, f.dim())))


def _solve(U, b, kappa, bc):
    """CG on the normal equations of the full operator, to 2e-14 |b|."""
    x = torch.zeros_like(b)
    r = b.clone()
    z = _dirac(U, r, kappa, bc, True)
    p, zz, bb = z.clone(), _norm2(z), _norm2(b)
    col = (slice(None),) + (None,) * (b.dim() - 1)
    for it in range(4000):
        q = _dirac(U, p, kappa, bc, False)
        a = zz / _norm2(q).clamp_min(1e-300)
        x += a[col] * p
        if it % 50 == 49:
            r = b - _dirac(U, x, kappa, bc, False)
        else:
            r -= a[col] * q
        if it % 10 == 9 and bool((_norm2(r) <= (2e-14) ** 2 * bb).all()):
            break
        z = _dirac(U, r, kappa, bc, True)
        zn = _norm2(z)
        p = z + (zn / zz.clamp_min(1e-300))[col] * p
        zz = zn
    return x


def _smear(U, psi, alpha, n, norm):
    for _ in range(n):
        h = torch.zeros_like(psi)
        for mu in range(3):
            ax = 4 - mu
            h += _umul(U[mu], torch.roll(psi, -1, ax), False)
            h += torch.roll(_umul(U[mu], psi, True), 1, ax)
        psi = (psi + alpha * h) / norm
    return psi


def _dag(m):
    return m.transpose(-1, -2).conj()


def _inv_dag(m):
    """(m^-1)^+ of 3x3 matrices: conj(cofactors) / conj(det)."""
    c = torch.stack([torch.linalg.cross(m[..., (i + 1) % 3, :], m[..., (i + 2) % 3, :]) for i in range(3)], dim=-2)
    det = (m[..., 0, :] * c[..., 0, :]).sum(-1)
    return (c / det[..., None, None]).conj(), det


def _ape(U, alpha, n):
    """APE steps of the spatial links, projected to SU(3) by the polar factor."""
    U = U.clone()
    for _ in range(n):
        new = []
        for i in range(3):
            acc = U[i].clone()
            for j in range(3):
                if j == i:
                    continue
                ai, aj = 3 - i, 3 - j  # axis of direction mu in [T][Z][Y][X] is 3 - mu
                acc += alpha * _mm(_mm(U[j], torch.roll(U[i], -1, aj)), _dag(torch.roll(U[j], -1, ai)))
                low = _mm(_mm(_dag(U[j]), U[i]), torch.roll(U[j], -1, ai))
                acc += alpha * torch.roll(low, 1, aj)
            for _k in range(30):
                inv, _d = _inv_dag(acc)
                nxt = 0.5 * (acc + inv)
                done = float((nxt - acc).abs().max()) < 1e-15
                acc = nxt
                if done:
                    break
            det = _inv_dag(acc)[1]
            new.append(acc * torch.exp(-1j * torch.angle(det) / 3)[..., None, None])
        U[:3] = torch.stack(new)
    return U


def _phases(mom, dims):
    """exp(2 pi i n.x / L) [nmom][Vs]."""
    z, y, x = torch.meshgrid(*[torch.arange(L, dtype=torch.float64, device=DEV) for L in (dims[2], dims[1], dims[0])],
                             indexing="ij")
    rows = []
    for a, b, c in mom:
        t = torch.remainder(a * x / dims[0] + b * y / dims[1] + c * z / dims[2], 1.0)
        rows.append(torch.polar(torch.ones_like(t), 2 * math.pi * t).reshape(-1))
    return torch.stack(rows)


def _project(L, mom, dims):
    """[ngamma][nmom][nt]"""
    ph = _phases(mom, dims)
    return torch.stack([(L * ph[k]).sum(-1) for k in range(len(mom))], dim=1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("exact", "stochastic", "tsm", "grad"):  # thousands of solves
        return None
    if case["kind"] == "solve" and case["nrhs"] * _vol(_dims(case["lattice"])) > 12 * 131072:
        return None
    x = _inputs(case, seed)
    dims = x["dims"][0]
    if kind == "corr":
        mom = MOM[: case["nmom"]]
        p1 = _project(x["L1"], mom, dims)
        p2 = _project(x["L2"], [(-a, -b, -c) for a, b, c in mom], dims)
        T = dims[3]
        d = torch.stack([(torch.roll(p1, -t, 2) * p2).sum(-1) for t in range(T)], dim=-1)
        return p1, p2, d / (_vol(dims[:3]) * T)
    U = _grid(x["U"][0], dims, 1)
    if kind == "pion":
        y0 = x["y0"]
        b = torch.zeros((12, _vol(dims), 4, 3), dtype=torch.complex128, device=DEV)
        for k in range(12):
            b[k, y0, k // 3, k % 3] = 1.0
        W = _ape(U, 0.5, case["ape"])
        norm = 1.0 + 6.0 * case["alpha"]
        b = _smear(W, _grid(b, dims, 1), case["alpha"], case["n"], norm)
        phi = _smear(W, _solve(U, b, case["kappa"], -1), case["alpha"], case["n"], norm)
        rho = phi.abs().square().sum(dim=(0, 5, 6)).reshape(1, dims[3], -1).to(torch.complex128)
        Vs = _vol(dims[:3])
        ph0 = _phases(MOM[:7], dims)[:, y0 % Vs].conj()
        return torch.roll(_project(rho, MOM[:7], dims)[0] * ph0[:, None], -(y0 // Vs), 1)
    psi = _grid(x["psi"], dims, 1)
    if kind == "apply":
        out = _dirac(U, psi, case["kappa"], -1, case["dagger"])
    elif kind == "smear":
        out = _smear(U, psi, case["alpha"], case["n"], 1.0 + 6.0 * case["alpha"])
    else:
        out = _solve(U, psi, case["kappa"], -1)
    return out.reshape(x["psi"].shape)
