"""The work this library is used for, as cases that can be timed through its public calls.

A case is a dict of plain values. ``prepare`` builds what a user's program holds before the
call (a context with a gauge field, packed sources, momenta, solver options), ``run`` makes
one pass through the public entry points and returns the whole outputs, ``work`` counts the
bytes and operations the pass cannot do without, and ``exact`` gives the same outputs in 64
bits from plain torch.

Inputs follow the recipe of the ``synth`` package (links exp(i eps H), Gaussian sources and
momenta, noise with density exp(-|xi|^2)), drawn on the GPU from the seed. Lattices are
written "L0xL1xL2xL3" (x0 first). ``tune`` says whether the program ran the library's hop
autotuner once after loading its gauge field, as the benchmark does, or uses the defaults,
as the tests do.
"""
import math

import torch

import paper_0710_0066_amd as sap

PREC = {"f64": sap.SAP_F64, "f32": sap.SAP_F32, "f16": sap.SAP_F16}
REAL = {"f64": 8, "f32": 4, "f16": 2}
METHOD = {"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB, "geom": sap.SAP_GEOM, "sap": sap.SAP_SAP_BICGSTAB}
COLOR = {"all": sap.SAP_ALL, "black": sap.SAP_BLACK, "white": sap.SAP_WHITE}
INNER_TOL = {"f64": 0.0, "f32": 1e-5, "f16": 2e-3}
EPS = 0.35                # link roughness of the named workloads
BETA = 5.6
FLOP_HOP = 1320           # one hop sum per output site and right-hand side
# operator applications (two half hops each) of one solve, rounded from the iteration
# counts of these solvers on these fields: what a solve to the given residual takes
APPLIES = {"cg": 300, "bicgstab": 150, "geom": 250, "sap": 120}


def listed():
    return [
        # one half hop and its partner on the smallest lattice (smoke runs, dense checks):
        # launch latency only
        dict(name="hop_4x4x4x4_f64", kind="hop", L="4x4x4x4", l0=2, kappa=0.155, nrhs=1, prec="f64", tune=False),
        # the full operator in FP64 on the plain workload, as a residual check calls it
        dict(name="M_32x16x16x16_f64", kind="M", L="32x16x16x16", l0=4, kappa=0.1575, nrhs=1, prec="f64", tune=False),
        # the black blocks of a lattice whose slices are not whole 64-site tiles, an odd
        # number of right-hand sides, FP32
        dict(name="W_24x10x6x14_f32_5rhs", kind="W", L="24x10x6x14", l0=6, kappa=0.15, nrhs=5, prec="f32",
             color="black", tune=False),
        # the benchmark's operator: the even-odd hop on 12 right-hand sides in FP32
        dict(name="hop_48x24x24x24_f32_12rhs", kind="hop", L="48x24x24x24", l0=4, kappa=0.158, nrhs=12, prec="f32",
             tune=True),
        # one propagator column: full-lattice solve, FP32 inner CG, the library's defaults
        dict(name="solve_32x16x16x16_cg_f32", kind="solve", L="32x16x16x16", l0=4, kappa=0.1575, nrhs=1, method="cg",
             inner="f32", tol=1e-11, tune=False),
        # the Schwarz-preconditioned solver of the paper's last action part
        dict(name="solve_32x16x16x16_sap", kind="solve", L="32x16x16x16", l0=4, kappa=0.14, nrhs=1, method="sap",
             inner="f64", tol=1e-11, tune=False),
        # the benchmark's batched block solves: every 24^3 x 4 block and 12 right-hand sides
        dict(name="blocks_48x24x24x24_cg_f32_12rhs", kind="blocks", L="48x24x24x24", l0=4, kappa=0.158, nrhs=12,
             level=1, method="cg", inner="f32", tol=1e-11, tune=True),
        # the same with the inner solver that is fastest there, FP16 storage, on one level below
        dict(name="blocks_48x24x24x24_bicgstab_f16_12rhs", kind="blocks", L="48x24x24x24", l0=4, kappa=0.158, nrhs=12,
             level=2, method="bicgstab", inner="f16", tol=1e-11, tune=True),
        # the pseudo-fermion force of the block action (two block solves and the force kernel)
        dict(name="pf_force_32x16x16x16", kind="pf_force", L="32x16x16x16", l0=4, kappa=0.1575, nrhs=1, method="cg",
             inner="f32", tol=1e-12, tune=False),
        # a short pure-gauge evolution: load a configuration, leap-frog steps, store it
        dict(name="gauge_md_48x24x24x24", kind="md", L="48x24x24x24", l0=4, kappa=0.158, steps=4, tune=False),
        # a short two-level trajectory of the two-factor action, the whole call
        dict(name="hmc_32x16x16x16", kind="hmc2", L="32x16x16x16", l0=4, kappa=0.1575, n_outer=2, n_inner=4, tau=0.1,
             tune=False),
        # a short five-level trajectory of the four-part action with the paper's solvers
        dict(name="hmc4_16x8x8x8", kind="hmc4", L="16x8x8x8", l0=8, l0_sub=4, kappa=0.13, n_outer=2, n_inner=2,
             tau=0.1, tune=False),
    ]


def draw(rng):
    """One more case: the same calls over the lattices, block lengths, right-hand sides,
    precisions and solvers between the listed ones."""
    def even(lo, hi):
        return 2 * max(lo // 2, min(hi // 2, round(math.exp(rng.uniform(math.log(lo / 2), math.log(hi / 2))))))

    def lattice(smax, blocks=(2, 3, 4, 5, 6)):
        l0 = rng.choice(blocks)
        L0 = 2 * l0 * rng.randint(1, max(1, 48 // (2 * l0)))
        return l0, "x".join(str(n) for n in (L0, even(4, smax), even(4, smax), even(4, smax)))

    kind = rng.choice(["hop", "M", "W", "solve", "blocks", "pf_force", "md", "hmc2", "hmc4"])
    c = dict(kind=kind, tune=rng.random() < 0.4)
    if kind in ("hop", "M", "W"):
        c["l0"], c["L"] = lattice(24)
        c.update(kappa=round(rng.uniform(0.12, 0.158), 4), prec=rng.choice(["f64", "f32", "f32", "f16"]),
                 nrhs=round(math.exp(rng.uniform(0, math.log(12)))))
        if kind == "W":
            c["color"] = rng.choice(["all", "black", "white"])
    elif kind in ("solve", "blocks"):
        c["l0"], c["L"] = lattice(16, (2, 4) if kind == "solve" else (4, 6, 8))
        c.update(nrhs=rng.choice([1, 1, 2, 3, 6, 12]), inner=rng.choice(["f64", "f32", "f32", "f16"]), tol=1e-11,
                 method=rng.choice(["cg", "bicgstab", "geom", "sap"] if kind == "solve" else
                                   ["cg", "bicgstab", "geom"]))
        c["kappa"] = round(rng.uniform(0.12, 0.1575 if c["method"] == "cg" else 0.135), 4)
        if kind == "blocks":
            c["level"] = rng.choice([1, 2])
            c["l0_sub"] = {4: 2, 6: 3, 8: 4}[c["l0"]]
    elif kind == "pf_force":
        c["l0"], c["L"] = lattice(16, (2, 4, 6))
        c.update(nrhs=1, method=rng.choice(["cg", "bicgstab"]), inner=rng.choice(["f64", "f32", "f32", "f16"]),
                 tol=1e-12)
        c["kappa"] = round(rng.uniform(0.12, 0.1575 if c["method"] == "cg" else 0.135), 4)
    elif kind == "md":
        c["l0"], c["L"] = lattice(24)
        c.update(kappa=0.15, steps=rng.randint(1, 6))
    else:
        L0 = rng.choice([8, 16])
        c["L"] = "x".join(str(n) for n in (L0, even(4, 10), even(4, 10), even(4, 10)))
        c.update(l0=4 if kind == "hmc2" else L0 // 2, kappa=round(rng.uniform(0.12, 0.135), 4), n_outer=rng.randint(1, 2),
                 n_inner=rng.choice([2, 4]) if kind == "hmc2" else 2, tau=round(rng.uniform(0.05, 0.12), 3))
        if kind == "hmc4":
            c["l0_sub"] = c["l0"] // 2
    return c


# ---- inputs -------------------------------------------------------------------------------

def dims(case):
    return tuple(int(n) for n in case["L"].split("x"))


def level2(case):
    """Level-2 block length: given, or half of l0 where that is a valid block length."""
    if "l0_sub" in case:
        return case["l0_sub"]
    return case["l0"] // 2 if case["l0"] % 4 == 0 else 0


def generator(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + k)
    return g


def gaussian(shape, gen, scale=1.0):
    x = torch.randn(tuple(shape) + (2,), generator=gen, dtype=torch.float64, device="cuda")
    return torch.view_as_complex(x.mul_(scale))


def mul3(a, b):
    """Products of stacks of 3 x 3 (or 3 x n) matrices, written out over the inner index."""
    return a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :] + a[..., :, 2:3] * b[..., 2:3, :]


def expm_i(H):
    """exp(i H) of Hermitian 3 x 3 stacks: Taylor series of exp(i H / 16), squared four times."""
    A = H * (1j / 16)
    one = torch.eye(3, dtype=A.dtype, device=A.device)
    E = one + A / 14
    for n in range(13, 0, -1):
        E = one + mul3(A, E) / n
    for _ in range(4):
        E = mul3(E, E)
    return E


def on_su3(U):
    """Rows orthonormalised, the third row the conjugate cross product of the first two."""
    a, b = U[..., 0, :], U[..., 1, :]
    a = a / a.abs().square().sum(-1, keepdim=True).sqrt()
    b = b - a * (a.conj() * b).sum(-1, keepdim=True)
    b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([a, b, torch.linalg.cross(a, b).conj()], dim=-2)


def gauge_field(L, gen):
    """Independent links exp(i EPS H), H = (A + A^+)/2 less its trace, A Gaussian."""
    U = torch.empty(tuple(L) + (4, 3, 3), dtype=torch.complex128, device="cuda")
    for mu in range(4):
        A = gaussian(tuple(L) + (3, 3), gen)
        H = (A + A.transpose(-1, -2).conj()) / 2
        H = H - torch.eye(3, device="cuda") * (torch.diagonal(H, dim1=-2, dim2=-1).sum(-1).real / 3)[..., None, None]
        U[:, :, :, :, mu] = on_su3(expm_i(EPS * H))
    return U


def solver_options(case, tol=None):
    kw = dict(tol=tol or case["tol"], max_iter=200000, inner_prec=PREC[case["inner"]], inner_tol=INNER_TOL[case["inner"]],
              max_outer=60, method=METHOD[case["method"]])
    if case["method"] == "sap":
        kw.update(sap_ncy=2, sap_block_terms=8)
    return sap.solve_opts(**kw)


def fields(case, seed):
    """The canonical inputs of a case: links, then sources, noise and momenta as it needs them."""
    L, kind = dims(case), case["kind"]
    f = {"U": gauge_field(L, generator(seed, 1))}
    if kind in ("hop", "M", "W", "solve", "blocks"):
        f["psi"] = gaussian((case["nrhs"],) + L + (4, 3), generator(seed, 2))
    elif kind == "pf_force":
        f["psi"] = gaussian((1,) + L + (4, 3), generator(seed, 2))
    if kind in ("md", "hmc2", "hmc4"):
        f["p"] = torch.randn(L + (4, 8), generator=generator(seed, 3), dtype=torch.float64, device="cuda")
    if kind in ("hmc2", "hmc4"):
        f["xi"] = [gaussian(L + (4, 3), generator(seed, 4 + k), math.sqrt(0.5)) for k in range(2 if kind == "hmc2" else 4)]
    return f


def prepare(case, seed):
    L, kind, nrhs = dims(case), case["kind"], case.get("nrhs", 1)
    f = fields(case, seed)
    ctx = sap.Context(L, case["l0"], case["kappa"], l0_sub=level2(case), max_rhs=nrhs)
    ctx.set_gauge(f["U"])
    if case["tune"]:
        sap.sap_tune(ctx, nrhs)
    s = {"case": case, "ctx": ctx, "nrhs": nrhs}
    if kind in ("hop", "M", "W"):
        prec = PREC[case["prec"]]
        s["in"], s["out"], s["prec"] = ctx.new_field(nrhs, prec), ctx.new_field(nrhs, prec), prec
        ctx.pack_spinor(s["in"], f["psi"], nrhs, prec)
    elif kind in ("solve", "blocks", "pf_force"):
        s["b"], s["opts"] = ctx.new_field(nrhs), solver_options(case)
        ctx.pack_spinor(s["b"], f["psi"], nrhs)
        if kind == "pf_force":
            s["F"] = ctx.new_momenta()
        else:
            s["x"] = ctx.new_field(nrhs)
    else:
        s["U0"], s["U"] = f["U"], torch.empty_like(f["U"])
        s["p0"] = ctx.new_momenta()
        ctx.pack_momenta(s["p0"], f["p"])
        if kind == "md":
            s["p"] = torch.empty_like(s["p0"])
        elif kind == "hmc2":
            o = sap.solve_opts(tol=1e-12, max_iter=500000, inner_prec=sap.SAP_F32, inner_tol=1e-6, max_outer=80)
            s["prm"] = sap.hmc_params(BETA, case["tau"], case["n_outer"], case["n_inner"], s["p0"], *f["xi"], 0.0, o, o)
        else:
            # the paper's solvers: geometric series for the first three parts, Schwarz-
            # preconditioned BiCGstab for the last
            o = sap.solve_opts(tol=1e-12, max_iter=500000, inner_prec=sap.SAP_F32, inner_tol=1e-6, max_outer=80)
            geom = sap.solve_opts(tol=1e-12, max_iter=500000, inner_prec=sap.SAP_F32, inner_tol=1e-6, max_outer=80,
                                  method=sap.SAP_GEOM)
            last = sap.solve_opts(tol=1e-12, max_iter=2000, inner_prec=sap.SAP_F32, inner_tol=1e-6, max_outer=80,
                                  method=sap.SAP_SAP_BICGSTAB, sap_ncy=1, sap_block_terms=8)
            n = (case["n_inner"], 2, 1, 1, case["n_outer"])
            s["prm"] = sap.hmc4_params(BETA, case["tau"], 0.2, n, s["p0"], *f["xi"], 0.0, o, o,
                                       part_solve=[geom, geom, geom, last] * 2)
    return s


# ---- one pass -----------------------------------------------------------------------------

def run(s):
    case, ctx, nrhs, kind = s["case"], s["ctx"], s["nrhs"], s["case"]["kind"]
    if kind == "hop":           # odd sites from even ones, then even sites from odd ones
        sap.apply_Dslash_eo(ctx, s["out"], s["in"], nrhs, 1, s["prec"])
        sap.apply_Dslash_eo(ctx, s["out"], s["in"], nrhs, 0, s["prec"])
        return stored(ctx, s["out"], nrhs, case["prec"])
    if kind == "M":
        sap.apply_M(ctx, s["out"], s["in"], nrhs, s["prec"])
        return stored(ctx, s["out"], nrhs, case["prec"])
    if kind == "W":
        sap.apply_W1_block(ctx, s["out"], s["in"], nrhs, 1, -1, COLOR[case["color"]], s["prec"])
        return stored(ctx, s["out"], nrhs, case["prec"])
    if kind == "solve":
        sap.solve_full(ctx, s["x"], s["b"], nrhs, s["opts"])
        return s["x"]
    if kind == "blocks":
        sap.solve_blocks(ctx, s["x"], s["b"], nrhs, case["level"], sap.SAP_ALL, s["opts"])
        return s["x"]
    if kind == "pf_force":
        s["F"].zero_()
        S = sap.block_pf_force(ctx, s["F"], 1.0, s["b"], s["opts"])
        return {"F": s["F"], "S": S}
    if kind == "md":
        dt = MD_DT
        ctx.set_gauge(s["U0"])
        s["p"].copy_(s["p0"])
        actions = []
        for _ in range(case["steps"]):
            actions.append(sap.gauge_force(ctx, s["p"], -0.5 * dt, BETA))
            sap.sap_update_links(ctx, s["p"], dt)
            actions.append(sap.gauge_force(ctx, s["p"], -0.5 * dt, BETA))
        ctx.get_gauge(s["U"])
        return {"U": s["U"], "p": s["p"], "S": torch.tensor(actions, dtype=torch.float64)}
    s["U"].copy_(s["U0"])
    info = (sap.hmc_trajectory if kind == "hmc2" else sap.hmc_trajectory_4pf)(ctx, s["U"], s["prm"])
    return {"U": s["U"], "H0": info.H0, "H1": info.H1, "plaq": info.plaq}


MD_DT = 0.02


def stored(ctx, out, nrhs, prec):
    """A field as it is stored: FP16 fields hold half-precision components and FP32 site norms."""
    if prec != "f16":
        return out
    w = out.view(nrhs, 26, -1)
    return {"components": w[:, :24].view(torch.float16), "norms": w[:, 24:]}


# ---- what a pass cannot do without --------------------------------------------------------

def work(case):
    L, kind, nrhs = dims(case), case["kind"], case.get("nrhs", 1)
    V = math.prod(L)
    site = lambda prec: 24 * REAL[prec] + (4 if prec == "f16" else 0)
    link = lambda prec: 4 * V * 18 * REAL[prec]
    if kind == "hop":           # links once, every site read and written once
        p = case["prec"]
        return {"bytes": link(p) + 2 * V * nrhs * site(p), "flops": FLOP_HOP * V * nrhs}
    if kind in ("M", "W"):
        p = case["prec"]
        part = 1.0 if kind == "M" or case["color"] == "all" else 0.5
        return {"bytes": part * link(p) + (1 + part) * V * nrhs * site(p), "flops": part * (FLOP_HOP + 48) * V * nrhs}
    if kind in ("solve", "blocks", "pf_force"):
        p, n = case["inner"], APPLIES[case["method"]] * (2 if kind == "pf_force" else 1)
        one = link(p) + 2 * V * nrhs * site(p)      # one operator application: two half hops
        ends = 2 * V * nrhs * site("f64") + link("f64")
        force = (72 * 8 + 2 * 192 + 512) * V if kind == "pf_force" else 0
        return {"bytes": n * one + ends + force, "flops": n * FLOP_HOP * V * nrhs}
    kick, move = 4 * V * (18 + 8 + 8) * 8, 4 * V * (18 + 8 + 18) * 8
    fkick, fmove = 4 * V * 13 * 216, 4 * V * 18 * 216
    if kind == "md":
        n = case["steps"]
        return {"bytes": (n + 1) * kick + n * move + 2 * link("f64"), "flops": (n + 1) * fkick + n * fmove}
    # trajectories: the solves of the force evaluations, heat baths and actions dominate
    kicks = 2 * case["n_outer"] + 1 if kind == "hmc2" else 12 * case["n_outer"]
    solves = 4 * kicks + 6 if kind == "hmc2" else 2 * kicks + 10
    per = APPLIES["cg"] if kind == "hmc2" else APPLIES["geom"] // 2
    return {"bytes": solves * per * (link("f32") + 2 * V * site("f32")), "flops": solves * per * FLOP_HOP * V}


# ---- the same in 64 bits, plain torch ------------------------------------------------------
# Spinors here are [rhs, L0, L1, L2, L3, spin, colour], links [L0, L1, L2, L3, mu, 3, 3].

GAMMA_ROWS = {            # gamma_mu psi: component s is phase * psi[source]
    0: [(2, -1), (3, -1), (0, -1), (1, -1)],
    1: [(3, -1j), (2, -1j), (1, 1j), (0, 1j)],
    2: [(3, -1), (2, 1), (1, 1), (0, -1)],
    3: [(2, -1j), (3, 1j), (0, 1j), (1, -1j)],
}


def gamma(mu, psi):
    return torch.stack([ph * psi[..., s, :] for s, ph in GAMMA_ROWS[mu]], dim=-2)


def gamma5(psi):
    return torch.cat([psi[..., :2, :], -psi[..., 2:, :]], dim=-2)


def colour(U, psi):
    """U psi per site on the colour index."""
    return sum(U[..., None, :, b] * psi[..., :, b, None] for b in range(3))


def dagger(U):
    return U.transpose(-1, -2).conj()


def shifted(psi, mu, step, l0):
    """psi(x + step mu), antiperiodic in x0; across x0 blocks of length l0 it is zero."""
    out = torch.roll(psi, -step, dims=1 + mu)
    if mu == 0:
        L0 = psi.shape[1]
        out[:, L0 - 1 if step > 0 else 0] *= -1
        if l0:
            edge = [x for x in range(L0) if x % l0 == (l0 - 1 if step > 0 else 0)]
            out[:, edge] = 0
    return out


def hop(U, psi, l0=0):
    out = torch.zeros_like(psi)
    for mu in range(4):
        f = colour(U[..., mu, :, :], shifted(psi, mu, 1, l0))
        out += f - gamma(mu, f)
        b = shifted(colour(dagger(U[..., mu, :, :]), psi), mu, -1, l0)
        out += b + gamma(mu, b)
    return out


def solve64(U, b, kappa, l0):
    """x with W x = b (l0 = 0: M), by conjugate gradients on the normal equations, restarted
    from the recomputed residual until that is at the rounding of 64 bits."""
    W = lambda v: v - kappa * hop(U, v, l0)
    Wd = lambda v: gamma5(W(gamma5(v)))
    dot = lambda v: v.abs().square().sum(dim=(1, 2, 3, 4, 5, 6), keepdim=True)
    x, bb = torch.zeros_like(b), dot(b)
    for _ in range(6):
        r = b - W(x)
        if bool((dot(r) <= 1e-27 * bb).all()):
            break
        s, e = r, torch.zeros_like(x)
        g = Wd(s)
        p, gg, r0 = g, dot(g), dot(r)
        for it in range(3000):
            q = W(p)
            a = gg / dot(q).clamp_min(1e-300)
            e = e + a * p
            s = s - a * q
            if it % 10 == 0 and bool((dot(s) <= 1e-20 * r0).all()):
                break
            g = Wd(s)
            new = dot(g)
            p = g + (new / gg.clamp_min(1e-300)) * p
            gg = new
        x = x + e
    return x


def parity_sites(L):
    """Lexicographic indices of the even, then of the odd sites."""
    grids = torch.meshgrid(*[torch.arange(n, device="cuda") for n in L], indexing="ij")
    par = (sum(grids) % 2).reshape(-1)
    return [torch.nonzero(par == p).reshape(-1) for p in (0, 1)]


def tiled(values, L, group):
    """[rhs, V, comps] -> the library's layout [rhs, parity, tile, comps / group, 64, group]."""
    n, V, comps = values.shape
    Vhp = (V // 2 + 63) // 64 * 64
    out = torch.zeros((n, 2, Vhp, comps), dtype=values.dtype, device=values.device)
    for p, idx in enumerate(parity_sites(L)):
        out[:, p, :V // 2] = values[:, idx]
    return out.view(n, 2, Vhp // 64, 64, comps // group, group).permute(0, 1, 2, 4, 3, 5).contiguous()


def stored64(psi, L, prec):
    v = psi.reshape(psi.shape[0], -1, 12)
    if prec != "f16":
        return torch.view_as_real(tiled(v, L, 2 if prec == "f32" else 1)).reshape(-1)
    r = torch.view_as_real(v)
    norm = r.abs().amax(dim=(2, 3))
    comps = tiled(v / norm.clamp_min(1e-300)[..., None], L, 4)
    n = psi.shape[0]
    norms = tiled(norm[..., None], L, 1).reshape(n, 2, -1)
    return {"components": torch.view_as_real(comps).reshape(n, 24, -1), "norms": norms}


def gell_mann():
    l = torch.zeros((8, 3, 3), dtype=torch.complex128)
    for a, (i, j) in zip((0, 3, 5), ((0, 1), (0, 2), (1, 2))):
        l[a, i, j] = l[a, j, i] = 1
        l[a + 1, i, j], l[a + 1, j, i] = -1j, 1j
    l[2] = torch.diag(torch.tensor([1, -1, 0], dtype=torch.complex128))
    l[7] = torch.diag(torch.tensor([1, 1, -2], dtype=torch.complex128)) / math.sqrt(3)
    # order lambda_1 .. lambda_8
    return l.cuda()


def im_tr(Q):
    """Im tr(lambda^a Q) for a = 1..8."""
    return torch.stack([(g.T * Q).sum(dim=(-1, -2)).imag for g in gell_mann()], dim=-1)


def outer(v, w):
    """sum over spin of v (x) w^*."""
    return sum(v[..., s, :, None] * w[..., s, None, :].conj() for s in range(4))


def pair_force64(U, a, b, kappa, l0):
    """2 Re <a, dW b> along U -> exp(i w T^a) U per link (one right-hand side each)."""
    F = torch.zeros(U.shape[:4] + (4, 8), dtype=torch.float64, device=U.device)
    for mu in range(4):
        Um = U[..., mu, :, :]
        bf, af = shifted(b, mu, 1, l0)[0], shifted(a, mu, 1, l0)[0]
        # -kappa <a, (1 - g) i T U b(x + mu)> + kappa <a(x + mu), (1 + g) i U^+ T b>
        X = outer(bf - gamma(mu, bf), a[0])
        Y = outer(b[0] + gamma(mu, b[0]), af)
        Q = mul3(Um, X) - mul3(Y, dagger(Um))
        F[..., mu, :] = kappa * im_tr(Q)
    return F


def roll(U, mu, step):
    return torch.roll(U, -step, dims=mu)


def staple_force64(U, beta):
    """dS_G/dw per link, and S_G."""
    F = torch.zeros(U.shape[:4] + (4, 8), dtype=torch.float64, device=U.device)
    total = 0.0
    for mu in range(4):
        A = torch.zeros_like(U[..., 0, :, :])
        Um = U[..., mu, :, :]
        for nu in range(4):
            if nu == mu:
                continue
            Un = U[..., nu, :, :]
            A += mul3(mul3(roll(Un, mu, 1), dagger(roll(Um, nu, 1))), dagger(Un))
            A += roll(mul3(mul3(dagger(roll(Un, mu, 1)), dagger(Um)), Un), nu, -1)
        W = mul3(Um, A)
        F[..., mu, :] = beta / 6 * im_tr(W)
        total += float(torch.diagonal(W, dim1=-2, dim2=-1).sum().real)
    return F, -beta / 3 * total / 4


def exact(case, seed):
    L, kind, kappa = dims(case), case["kind"], case["kappa"]
    V = math.prod(L)
    if kind in ("hmc2", "hmc4"):
        return None           # a whole trajectory of solves takes too long here
    if kind in ("solve", "blocks") and V * case["nrhs"] > 600000:
        return None
    f = fields(case, seed)
    U = f["U"]
    if kind in ("hop", "M", "W"):
        l0 = case["l0"] if kind == "W" else 0
        outs = []
        for psi in f["psi"].split(1):
            D = hop(U, psi, l0)
            v = D if kind == "hop" else psi - kappa * D
            if kind == "W" and case["color"] != "all":
                for x in range(L[0]):
                    if (x // l0) % 2 != (1 if case["color"] == "black" else 0):
                        v[:, x] = 0
            outs.append(v)
        return stored64(torch.cat(outs), L, case["prec"])
    if kind in ("solve", "blocks"):
        l0 = 0 if kind == "solve" else case["l0"] if case["level"] == 1 else level2(case)
        return stored64(solve64(U, f["psi"], kappa, l0), L, "f64")
    if kind == "pf_force":
        X = solve64(U, f["psi"], kappa, case["l0"])
        Y = gamma5(solve64(U, gamma5(X), kappa, case["l0"]))
        F = -pair_force64(U, Y, X, kappa, case["l0"])
        return {"F": tiled(F.reshape(1, V, 32), L, 1).reshape(-1), "S": float(X.abs().square().sum())}
    p, S = f["p"], []
    T = gell_mann() / 2
    force, action = staple_force64(U, BETA)
    for _ in range(case["steps"]):
        S.append(action)
        p = p - 0.5 * MD_DT * force
        for mu in range(4):
            P = sum(p[..., mu, a, None, None] * T[a] for a in range(8))
            U[..., mu, :, :] = on_su3(mul3(expm_i(MD_DT * P), U[..., mu, :, :]))
        force, action = staple_force64(U, BETA)
        S.append(action)
        p = p - 0.5 * MD_DT * force
    return {"U": U, "p": tiled(p.reshape(1, V, 32), L, 1).reshape(-1), "S": torch.tensor(S, dtype=torch.float64)}
