"""Performance cases of the exact-exchange / ACE library: the calls a user's
program makes in earnest, with inputs of the repository's own recipes.

A case's "kind" names the call sequence:

  exx    sea.Context.exx_action on one cell (pair solves, W, E_xx); cube pair
         domains ("rule": "cube") or the epsilon-driven ones with their W
         boxes ("eps"); CG state and start as the options say
  plan   the same action of several cells replayed from a HIP-graph plan
  chain  sea.Context.build_pairs_eps, then exx_action on those pairs: one outer
         iteration whose orbitals, and so whose boxes, are new
  ace    ace_build, ace_apply on trial vectors and ace_energy
  apply  ace_apply alone (the repeated product of an outer SCF loop)
  scdm   scdm of delocalized orbitals and the back-rotation of W
  train  one training step of the start network (forward, backward, Adam)

Cells are the seeded water-like ones (4 orbitals per molecule); the grid
spacing is the production one (0.196 bohr) unless a case gives "N".
"""
import math
import os

import numpy as np
import torch

from paper_2208_06097_amd import sea, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WEIGHTS = os.path.join(ROOT, "paper_2208_06097_amd", "weights", "unet_f32cg.npy")
EPS = 10 ** -3.5          # the paper's production setting of the epsilon rule
DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
SEA_DTYPES = {"f64": sea.SEA_F64, "f32": sea.SEA_F32, "bf16": sea.SEA_BF16}
STARTS = {"zero": sea.SEA_START_ZERO, "multipole": sea.SEA_START_MULTIPOLE, "learned": sea.SEA_START_LEARNED,
          "spectral": sea.SEA_START_SPECTRAL}


def listed():
    return [
        # the smallest call: a few-molecule cell with the library's default
        # options (FP64 CG from zero), host results returned; launches and
        # host round trips count
        dict(name="exx-3mol-default", kind="exx", n_mol=3, L=9.0, N=30, half=4.0, rule="cube", phi="f64",
             state="f64", start="zero", host=True, tune=False),
        # the 8-molecule cell (60^3 grid, domains wider than the cell), the
        # form used for production actions
        dict(name="exx-8mol-spectral", kind="exx", n_mol=8, L=11.7, N=60, half=6.0, rule="cube", phi="f64",
             state="f32", start="spectral", host=False, tune=False),
        # the same cell through the FP32 CG from the learned start (network
        # inference, FP32 state with FP64 reliable updates)
        dict(name="exx-8mol-learned", kind="exx", n_mol=8, L=11.7, N=60, half=6.0, rule="cube", phi="f64",
             state="f32", start="learned", host=False, tune=False),
        # the 64-molecule cell at 1.0 g/cm^3 (120^3, 256 orbitals): the
        # benchmark's action, schedules tuned once as the benchmark does
        dict(name="exx-64mol-spectral", kind="exx", n_mol=64, L=23.5, N=120, half=6.0, rule="cube", phi="f64",
             state="f32", start="spectral", host=False, tune=True),
        # the paper's own truncation on that cell: ragged boxes of every
        # parity, W on the Omega^D boxes, statistics returned
        dict(name="exx-64mol-eps", kind="exx", n_mol=64, L=23.5, N=120, half=6.0, rule="eps", phi="f64",
             state="f32", start="spectral", host=True, tune=False),
        # batching: two cells of different density, FP32 orbitals, replayed
        # from one graph plan as the batch driver does
        dict(name="plan-2x27mol-f32", kind="plan", n_cells=2, n_mol=27, rho=0.7, rho_step=0.6, phi="f32",
             start="spectral"),
        # an outer iteration with new orbitals on that cell: box search,
        # screening and W boxes, then the action on them
        dict(name="chain-64mol", kind="chain", n_mol=64, L=23.5, N=120, phi="f64", start="spectral"),
        # the benchmark step's ACE part: M and Cholesky in FP64, xi and K psi
        # in FP32, 256 trial vectors, the Eq. 19 energy
        dict(name="ace-64mol-f32", kind="ace", n_mol=64, L=23.5, N=120, dtype="f32", n_vec=256),
        # the same in FP64 on a small cell with few trial vectors
        dict(name="ace-8mol-f64", kind="ace", n_mol=8, L=11.7, N=60, dtype="f64", n_vec=20),
        # K psi alone in BF16, ragged orbital and vector counts and an odd grid
        dict(name="apply-38mol-bf16", kind="apply", n_mol=38, L=19.8, N=101, dtype="bf16", n_vec=200),
        # SCDM localization of the 64-molecule cell's delocalized orbitals and
        # the rotation of W back to them
        dict(name="scdm-64mol", kind="scdm", n_mol=64, L=23.5, N=120, dtype="f64"),
        # one step of the trainer at its batch size, learning rate at the end
        # of its schedule
        dict(name="train-b32", kind="train", batch=32, D=32, weights="bf16"),
    ]


def _loguniform(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def _cell_sizes(rng, n_mol_max, rho=(0.6, 1.6)):
    """Molecules, cell side and grid points of a cell at the production spacing."""
    n_mol = min(n_mol_max, max(2, int(round(_loguniform(rng, 2, n_mol_max)))))
    L = round((n_mol / 64.0 / rng.uniform(*rho)) ** (1 / 3) * synth.REF_L, 2)
    return n_mol, L, int(round(L / synth.H_TARGET)) + rng.choice((0, 0, 1))


def draw(rng):
    kind = rng.choice(("exx", "exx", "exx", "eps", "plan", "chain", "ace", "apply", "scdm", "train", "default"))
    if kind == "default":
        n_mol = rng.randint(2, 4)
        return dict(kind="exx", n_mol=n_mol, L=round(rng.uniform(8.0, 10.0), 2), N=rng.randint(28, 40),
                    half=round(rng.uniform(3.6, 4.4), 2), rule="cube", phi=rng.choice(("f64", "f32")), state="f64",
                    start=rng.choice(("zero", "multipole")), host=True, tune=False)
    if kind == "exx":
        start = rng.choice(("spectral", "spectral", "spectral", "learned", "multipole"))
        n_mol, L, N = _cell_sizes(rng, 48 if start == "spectral" else 10)
        return dict(kind="exx", n_mol=n_mol, L=L, N=N, half=round(rng.uniform(4.0, 6.0), 2), rule="cube",
                    phi=rng.choice(("f64", "f32")), state="f32", start=start, host=rng.random() < 0.5, tune=False)
    if kind == "eps":
        n_mol, L, N = _cell_sizes(rng, 56)
        return dict(kind="exx", n_mol=n_mol, L=L, N=N, half=6.0, rule="eps", phi=rng.choice(("f64", "f32")),
                    state="f32", start="spectral", host=rng.random() < 0.5, tune=False)
    if kind == "plan":
        return dict(kind="plan", n_cells=rng.randint(1, 3), n_mol=rng.randint(4, 20), rho=round(rng.uniform(0.5, 0.9), 3),
                    rho_step=round(rng.uniform(0.1, 0.4), 3), phi=rng.choice(("f32", "f64")), start="spectral")
    if kind == "chain":
        n_mol, L, N = _cell_sizes(rng, 56)
        return dict(kind="chain", n_mol=n_mol, L=L, N=N, phi=rng.choice(("f64", "f32")), start="spectral")
    if kind in ("ace", "apply"):
        n_mol, L, N = _cell_sizes(rng, 56)
        return dict(kind=kind, n_mol=n_mol, L=L, N=N, dtype=rng.choice(("f64", "f32", "bf16")),
                    n_vec=int(round(_loguniform(rng, 1, 4 * n_mol))))
    if kind == "scdm":
        n_mol, L, N = _cell_sizes(rng, 48)
        return dict(kind="scdm", n_mol=n_mol, L=L, N=N, dtype=rng.choice(("f64", "f64", "f32")))
    return dict(kind="train", batch=rng.randint(1, 40), D=rng.choice((16, 24, 32)), weights=rng.choice(("bf16", "f32")))


# ------------------------------------------------------------------ inputs

def _orbitals(case, seed, dtype):
    cell = synth.make_centres(case["n_mol"], case["L"], case["N"], seed)
    return cell, synth.fill_orbitals_device(cell, dtype=dtype)


def _plan_cells(case, seed):
    out = []
    for k in range(case["n_cells"]):
        L = (case["n_mol"] / 64.0 / (case["rho"] + k * case["rho_step"])) ** (1 / 3) * synth.REF_L
        cell = synth.make_centres(case["n_mol"], L, int(round(L / synth.H_TARGET)), seed + 1000 * k)
        out.append((cell, synth.fill_orbitals_device(cell, dtype=DTYPES[case["phi"]])))
    return out


def _context(case):
    ctx = sea.Context(stencil_dtype=SEA_DTYPES[case.get("state", "f32")], start=STARTS[case["start"]])
    if case["start"] == "learned":
        ctx.nn_attach(ctx.nn_state(np.load(WEIGHTS)))
    return ctx


def _potential(cell):
    """A smooth positive periodic potential on the grid: W = potential * phi
    has the shape of an exchange action (localized, M symmetric positive)."""
    c = torch.cos(2 * math.pi / cell.N * torch.arange(cell.N, dtype=torch.float64, device="cuda"))
    return 0.9 + 0.2 * c[:, None, None] + 0.15 * c[None, :, None] + 0.1 * c[None, None, :]


def _ace_inputs(case, seed):
    """(cell, phi, W, psi): orbitals, an action on them, trial vectors."""
    cell, phi = _orbitals(case, seed, torch.float64)
    W = phi * _potential(cell)
    other = synth.make_centres(max(case["n_mol"], -(-case["n_vec"] // 4)), case["L"], case["N"], seed + 1)
    other.centres, other.a = other.centres[:case["n_vec"]], other.a[:case["n_vec"]]
    return cell, phi, W, synth.fill_orbitals_device(other).to(DTYPES[case["dtype"]])


def _xi(cell, phi, W, dtype):
    """xi = W L^-T of the inputs (Eq. 18), in the case's type."""
    P, Wm = phi.flatten(1), W.flatten(1)
    M = cell.h ** 3 * (P @ Wm.T)
    return (_inverse_factor(M)[1] @ Wm).to(dtype).view(W.shape)


def _inverse_factor(M):
    """(L, L^-1) of the symmetrized M."""
    Lm = torch.linalg.cholesky((0.5 * (M + M.T)).cpu())
    return Lm.cuda(), torch.linalg.inv(Lm).cuda()


def _delocalized(case, seed):
    cell, phi = _orbitals(case, seed, torch.float64)
    G = torch.from_numpy(synth.random_rotation(cell.n_occ, seed + 7)).cuda()
    return cell, (G.T @ phi.flatten(1)).view_as(phi).to(DTYPES[case["dtype"]]).contiguous()


def _train_inputs(case, seed):
    """Inputs like the sampled pair densities (a few Gaussians of order-one
    mass on the D^3 grid) and smooth small targets."""
    g = torch.Generator().manual_seed(seed)
    B, D = case["batch"], case["D"]
    ax = torch.linspace(-6, 6, D, dtype=torch.float64)
    x = torch.zeros(B, D, D, D, dtype=torch.float64)
    t = torch.zeros_like(x)
    for out, width, scale in ((x, 0.8, 0.3), (t, 2.2, 0.05)):
        for _ in range(3):
            c = 1.5 * torch.randn(B, 3, generator=g, dtype=torch.float64)
            a = scale * torch.randn(B, generator=g, dtype=torch.float64)
            f = [torch.exp(-(ax[None] - c[:, k:k + 1]) ** 2 / (2 * width * width)) for k in range(3)]
            out += a[:, None, None, None] * f[0][:, :, None, None] * f[1][:, None, :, None] * f[2][:, None, None, :]
    return x.float().cuda(), t.float().cuda()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "exx":
        cell, phi = _orbitals(case, seed, DTYPES[case["phi"]])
        ctx = _context(case)
        dbox = None
        if case["rule"] == "eps":
            pairs, _, dbox = ctx.build_pairs_eps(phi, cell.N, cell.L, EPS, EPS, pad=6, with_dbox=True)
        else:
            pairs = sea.build_pairs(cell.N, cell.L, cell.centres, 6.0, case["half"])
        s = dict(kind=kind, ctx=ctx, phi=phi, N=cell.N, L=cell.L, pairs=pairs, dbox=dbox, host=case["host"])
        s["W"] = torch.empty(phi.shape, dtype=torch.float64, device="cuda")
        s["E"] = torch.zeros(1, dtype=torch.float64, device="cuda")
        if dbox is None:
            s["ws"] = ctx.workspace(ctx.exx_workspace_bytes(cell.N, cell.L, cell.n_occ, pairs))
        else:
            s["ws"] = ctx.workspace(ctx.exx_batched_workspace_bytes([(phi, cell.N, cell.L, pairs, s["W"], s["E"], dbox)]))
        if case["tune"]:
            ctx.spectral_autotune([(phi, cell.N, cell.L, pairs)], sample_pairs=2048, ws=s["ws"])
            ctx.scatter_autotune([(phi, cell.N, cell.L, pairs, s["W"])], ws=s["ws"])
        return s
    if kind == "plan":
        ctx = _context(case)
        cells, E = [], torch.zeros(case["n_cells"], dtype=torch.float64, device="cuda")
        for k, (cell, phi) in enumerate(_plan_cells(case, seed)):
            pairs = sea.build_pairs(cell.N, cell.L, cell.centres, 6.0, 6.0)
            cells.append((phi, cell.N, cell.L, pairs, torch.empty(phi.shape, dtype=torch.float64, device="cuda"), E[k:]))
        return dict(kind=kind, ctx=ctx, plan=ctx.exx_plan(cells), cells=cells, E=E)
    if kind == "chain":
        cell, phi = _orbitals(case, seed, DTYPES[case["phi"]])
        return dict(kind=kind, ctx=_context(case), phi=phi, N=cell.N, L=cell.L,
                    W=torch.empty(phi.shape, dtype=torch.float64, device="cuda"),
                    E=torch.zeros(1, dtype=torch.float64, device="cuda"))
    if kind in ("ace", "apply"):
        cell, phi, W, psi = _ace_inputs(case, seed)
        ctx = sea.Context(ace_dtype=SEA_DTYPES[case["dtype"]])
        ws = ctx.workspace(ctx.ace_workspace_bytes(cell.N ** 3, cell.n_occ, case["n_vec"]))
        s = dict(kind=kind, ctx=ctx, psi=psi, dV=cell.h ** 3, ws=ws)
        if kind == "ace":
            return s | dict(phi=phi, W=W)
        return s | dict(xi=_xi(cell, phi, W, DTYPES[case["dtype"]]))
    if kind == "scdm":
        cell, phi = _delocalized(case, seed)
        ctx = sea.Context()
        return dict(kind=kind, ctx=ctx, phi=phi, W=(phi * _potential(cell)).to(phi.dtype),
                    ws=ctx.workspace(ctx.scdm_workspace_bytes(cell.N ** 3, cell.n_occ)))
    x, t = _train_inputs(case, seed)
    ctx = sea.Context(nn_weight_dtype=SEA_DTYPES[case["weights"]])
    state = ctx.nn_state(np.load(WEIGHTS))
    grad = torch.empty(ctx.nn_param_count(), dtype=torch.float32, device="cuda")
    return dict(kind=kind, ctx=ctx, x=x, t=t, state=state, ws=ctx.nn_workspace(case["batch"], case["D"]), grad=grad,
                step=0)


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "exx":
        ctx.exx_action(s["phi"], s["N"], s["L"], s["pairs"], ws=s["ws"], W=s["W"], exx_dev=s["E"],
                       want_host=s["host"], dbox=s["dbox"])
        return {"W": s["W"], "E": s["E"]}
    if kind == "plan":
        s["plan"].launch()
        return {"W": s["plan"].W, "E": s["E"]}
    if kind == "chain":
        pairs, _, dbox = ctx.build_pairs_eps(s["phi"], s["N"], s["L"], EPS, EPS, pad=6, with_dbox=True)
        ctx.exx_action(s["phi"], s["N"], s["L"], pairs, W=s["W"], exx_dev=s["E"], want_host=False, dbox=dbox)
        return {"W": s["W"], "E": s["E"]}
    if kind == "ace":
        M, Lm, xi, _ = ctx.ace_build(s["phi"], s["W"], s["dV"], ws=s["ws"])
        Kpsi = ctx.ace_apply(xi, s["psi"], s["dV"], ws=s["ws"])
        return {"M": M, "L": Lm, "xi": xi, "Kpsi": Kpsi, "E": ctx.ace_energy(s["phi"], xi, s["dV"], ws=s["ws"])}
    if kind == "apply":
        return {"Kpsi": ctx.ace_apply(s["xi"], s["psi"], s["dV"], ws=s["ws"])}
    if kind == "scdm":
        r = ctx.scdm(s["phi"], ws=s["ws"])
        back = ctx.rotate(s["W"], r["U"], inverse=True)
        return {"U": r["U"], "loc": r["phi_loc"], "piv": r["piv"], "rdiag": r["rdiag"], "back": back}
    s["step"] += 1
    loss = ctx.nn_train_step(s["state"], s["x"], s["t"], 1e-6, s["step"], ws=s["ws"], grad=s["grad"])
    return {"loss": loss, "grad": s["grad"]}


# ------------------------------------------------------------------ work

def _expected_pairs(n_mol, L, reach):
    """Pairs of 4 n_mol orbitals closer than `reach` in a cell of side L."""
    n = 4 * n_mol
    near = min(1.0, 4 / 3 * math.pi * reach ** 3 / L ** 3)
    return n + 0.5 * n * (n - 1) * near


def _exx_work(n_mol, L, N, half, rule, phi):
    """Orbitals read and W written once; per pair-domain point about 100
    flops: six one-axis fast sine transforms, the division, rho, W and e_ij."""
    h = L / N
    n = 2 * math.ceil(half / h) + 1 if rule == "cube" else min(N, round(6.1 / h))
    pairs = _expected_pairs(n_mol, L, 6.0 if rule == "cube" else 4.2)
    return 4 * n_mol * N ** 3 * (8.0 + (8.0 if phi == "f64" else 4.0)), pairs * n ** 3 * 100.0


def work(case):
    kind = case["kind"]
    if kind == "exx":
        b, f = _exx_work(case["n_mol"], case["L"], case["N"], case["half"], case["rule"], case["phi"])
    elif kind == "plan":
        b = f = 0.0
        for k in range(case["n_cells"]):
            L = (case["n_mol"] / 64.0 / (case["rho"] + k * case["rho_step"])) ** (1 / 3) * synth.REF_L
            bk, fk = _exx_work(case["n_mol"], L, int(round(L / synth.H_TARGET)), 6.0, "cube", case["phi"])
            b, f = b + bk, f + fk
    elif kind == "chain":
        b, f = _exx_work(case["n_mol"], case["L"], case["N"], 6.0, "eps", case["phi"])
    elif kind in ("ace", "apply"):
        n, Ng, nv = 4 * case["n_mol"], float(case["N"] ** 3), case["n_vec"]
        w = {"f64": 8, "f32": 4, "bf16": 2}[case["dtype"]]
        wo = max(4, w)
        b, f = n * Ng * w + nv * Ng * (w + wo), 4.0 * n * nv * Ng
        if kind == "ace":   # phi and W in FP64, xi written; M, xi, energy products
            b, f = b + 16.0 * n * Ng, f + 2.0 * n * n * Ng * (0.5 + 0.5 + 1.0)
    elif kind == "scdm":
        n, Ng = 4 * case["n_mol"], float(case["N"] ** 3)
        w = 8 if case["dtype"] == "f64" else 4
        b, f = 4 * n * Ng * w, 4.0 * n * n * Ng
    else:
        v = case["batch"] * case["D"] ** 3
        levels = {0: (1 + 16 + 32 + 16) * 16 + 16, 1: (16 + 16 + 32 + 16) * 16, 2: (16 + 16 + 32 + 16) * 16,
                  3: (16 + 16) * 16}
        macs = sum(27 * c * v / 8 ** lv for lv, c in levels.items())
        b, f = 8.0 * v + 16 * 111681.0, 6.0 * macs
    return {"bytes": float(b), "flops": float(f)}


# ------------------------------------------------------------------ exact
# The same results from the definitions in 64 bits (plain torch and numpy).

LMAX = 6
FD = [-5369 / 1800, 12 / 7, -15 / 56, 10 / 189, -1 / 112, 2 / 1925, -1 / 16632]   # O(h^12) second derivative


def _harmonic_table():
    """Coefficients H[l*l+l+m][a, b, c] of the real solid harmonics
    (normalized so that 1/|r-r'| = sum R_lm(r') R_lm(r) / r^(2l+1)) in
    x^a y^b z^c."""
    n = LMAX + 1
    shift = lambda p, ax: np.roll(p, 1, axis=ax)  # noqa: E731   (degrees stay below n)
    one = np.zeros((n + 1,) * 3)
    one[0, 0, 0] = 1.0
    R = {(0, 0): one}
    for l in range(LMAX):
        c, s = R[(l, l)], R.get((l, -l), 0 * one) if l else 0 * one
        k = math.sqrt((2 * l + 1) / (2 * l + 2)) * (math.sqrt(2.0) if l == 0 else 1.0)
        R[(l + 1, l + 1)] = k * (shift(c, 0) - shift(s, 1))
        R[(l + 1, -l - 1)] = k * (shift(c, 1) + shift(s, 0))
        for m in range(-l, l + 1):
            p = (2 * l + 1) * shift(R[(l, m)], 2)
            if l - 1 >= abs(m):
                q = R[(l - 1, m)]
                p = p - math.sqrt((l + m) * (l - m)) * sum(shift(shift(q, ax), ax) for ax in range(3))
            R[(l + 1, m)] = p / math.sqrt((l + 1 + m) * (l + 1 - m))
    return np.stack([R[(l, m)][:n, :n, :n] for l in range(n) for m in range(-l, l + 1)])


class _PairSolver:
    """Direct solve of the discrete pair problem: the stencil matrix is a sum
    of one-axis matrices, so their eigenvectors diagonalize it."""

    def __init__(self, h):
        self.h = h
        self.H = torch.from_numpy(_harmonic_table()).cuda()
        self.lm = [l for l in range(LMAX + 1) for _ in range(2 * l + 1)]
        self.eig, self.tap = {}, {}

    def axis(self, n):
        if n not in self.eig:
            T = np.zeros((n, n))
            for k, c in enumerate(FD):
                T -= c * (np.eye(n, k=k) + (np.eye(n, k=-k) if k else 0)) / self.h ** 2 if k < n else 0
            lam, Q = np.linalg.eigh(T)
            G = np.zeros((min(n, 6), 6))
            for i in range(min(n, 6)):
                for j in range(6 - i):
                    G[i, j] = FD[i + j + 1] / self.h ** 2
            self.eig[n] = tuple(torch.from_numpy(v).cuda() for v in (lam, Q))
            self.tap[n] = torch.from_numpy(G).cuda()
        return self.eig[n]

    def powers(self, u):
        return torch.stack([u ** k for k in range(LMAX + 1)])

    def multipole(self, C, x, y, z):
        """sum_l P_l(r) / r^(2l+1) on the product grid (z, y, x)."""
        P = torch.tensordot(C, self.powers(z), dims=([3], [0]))          # l a b z
        P = torch.einsum("labz,by->lazy", P, self.powers(y))
        P = torch.einsum("lazy,ax->lzyx", P, self.powers(x))
        r2 = z[:, None, None] ** 2 + y[None, :, None] ** 2 + x[None, None, :] ** 2
        ir = torch.rsqrt(r2)
        out, f = 0.0, ir
        for l in range(LMAX + 1):
            out = out + P[l] * f
            f = f * ir * ir
        return out

    def __call__(self, rho, off):
        """rho on (z, y, x), `off`: displacement of the box's first point from
        the origin; returns (v, coefficients of the multipole sum)."""
        n = rho.shape[::-1]
        h = self.h
        ax = [off[a] + h * torch.arange(-6, n[a] + 6, dtype=torch.float64, device="cuda") for a in range(3)]
        ins = [u[6:-6] for u in ax]
        px, py, pz = (self.powers(u) for u in ins)
        mom = torch.einsum("zyx,ax->zya", rho, px)
        mom = torch.einsum("zya,by->zab", mom, py)
        mom = torch.einsum("zab,cz->abc", mom, pz) * h ** 3
        q = torch.einsum("kabc,abc->k", self.H, mom)
        C = torch.zeros((LMAX + 1,) * 4, dtype=torch.float64, device="cuda")
        C.index_add_(0, torch.tensor(self.lm, device="cuda"), self.H * q[:, None, None, None])
        b = 4 * math.pi * rho
        eig = [self.axis(k) for k in n]
        for a in range(3):
            m = min(n[a], 6)
            G = self.tap[n[a]]
            for side in (0, 1):
                gh = ax[a][:6].flip(0) if side == 0 else ax[a][-6:]       # nearest ghost layer first
                u = [gh if k == a else ins[k] for k in range(3)]
                d = torch.tensordot(G, self.multipole(C, *u), dims=([1], [2 - a]))
                d = d.movedim(0, 2 - a)
                if side == 0:
                    b.narrow(2 - a, 0, m).add_(d)
                else:
                    b.narrow(2 - a, n[a] - m, m).add_(d.flip(2 - a))
        v = b
        for a in range(3):
            v = torch.tensordot(v, eig[a][1], dims=([0 if a == 2 else 2 - a], [0])).movedim(-1, 2 - a)
        v = v / (eig[2][0][:, None, None] + eig[1][0][None, :, None] + eig[0][0][None, None, :])
        for a in range(3):
            v = torch.tensordot(v, eig[a][1], dims=([2 - a], [1])).movedim(-1, 2 - a)
        return v, C


def _cube_pairs(cell, half):
    """(i, j, lo, n, origin) of every pair closer than 6 bohr."""
    h, c = cell.h, cell.centres
    w = math.ceil(half / h - 1e-12)
    out = []
    for i in range(cell.n_occ):
        for j in range(i, cell.n_occ):
            d = c[j] - c[i]
            d = d - cell.L * np.rint(d / cell.L)
            if i == j or math.sqrt(float(d @ d)) < 6.0:
                k = np.floor((c[i] + 0.5 * d) / h + 0.5).astype(int)
                out.append((i, j, k - w, np.full(3, 2 * w + 1), k * h, None))
    return out


def _run_boxes(cell, phi):
    """Shortest cyclic runs of 1 - EPS/3 of each axis's marginal mass."""
    N = cell.N
    sq = [torch.stack([(p.double() ** 2).sum(dim=[k for k in range(3) if k != 2 - a]) for p in phi]).cpu().numpy()
          for a in range(3)]
    lo, ln = np.zeros((len(phi), 3), int), np.zeros((len(phi), 3), int)
    for i in range(len(phi)):
        for a in range(3):
            m = sq[a][i]
            cum = np.concatenate([[0.0], np.cumsum(np.concatenate([m, m]))])
            target = (1 - EPS / 3) * m.sum()
            ln[i, a] = N
            for k in range(1, N):
                mass = cum[k:k + N] - cum[:N]
                if mass.max() >= target:
                    lo[i, a], ln[i, a] = int(np.argmax(mass)), k
                    break
    return lo, ln


def _eps_pairs(cell, phi, pad):
    N, h = cell.N, cell.h
    lo, ln = _run_boxes(cell, phi)
    out = []

    def nearest(l, n, r0, rn):
        return min((l, l - N, l + N), key=lambda s: (abs(2 * s + n - 2 * r0 - rn), (l - N, l, l + N).index(s)))

    for i in range(len(phi)):
        for j in range(i, len(phi)):
            st, n = np.zeros(3, int), np.zeros(3, int)
            for a in range(3):
                p, lp, q, lq = lo[i, a], ln[i, a], lo[j, a], ln[j, a]
                if lp >= N or lq >= N:
                    st[a], n[a] = (q, lq) if lp >= N else (p, lp)
                    continue
                for k in (-1, 0, 1):
                    s, e = max(p, q + k * N), min(p + lp, q + k * N + lq)
                    if e - s > n[a]:
                        st[a], n[a] = s, e - s
            if n.min() <= 0:
                continue
            ix = [torch.arange(st[a], st[a] + n[a], device="cuda") % N for a in range(3)]
            at = (ix[2][:, None, None], ix[1][None, :, None], ix[0][None, None, :])
            S = h ** 3 * (phi[i][at].double() * phi[j][at].double()).abs().sum()
            out.append((i, j, st, n, S))
    keep = (torch.stack([o[4] for o in out]) >= EPS).cpu().numpy()
    pairs = []
    for i, j, st, n, _ in (o for o, k in zip(out, keep) if k):
        n2 = np.minimum(n + 2 * pad, N)
        l2 = st - (n2 - n) // 2
        db = []
        for o, partner in ((i, j), (j, i)):
            for_self = i == j and o == i and not db
            l = np.zeros(3, int)
            m = np.zeros(3, int)
            for a in range(3):
                if for_self:
                    m[a] = min(2 * ln[i, a], N)
                    s = lo[i, a] - (m[a] - ln[i, a]) // 2
                else:
                    m[a], s = ln[partner, a], lo[partner, a]
                s = nearest(s, m[a], l2[a], n2[a])
                e = max(s + m[a], l2[a] + n2[a])
                l[a] = min(s, l2[a])
                m[a] = min(e - l[a], N)
            db += [l, m]
        pairs.append((i, j, l2, n2, (l2 + 0.5 * (n2 - 1)) * h, db))
    return pairs


def _exx_exact(cell, phi, pairs):
    """(W, E) of Eq. 8-14."""
    N, h = cell.N, cell.h
    phi = phi.double()
    W = torch.zeros_like(phi)
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    solve = _PairSolver(h)
    grid = torch.arange(N, device="cuda")

    def index(lo, n):
        ix = [grid[(torch.arange(int(lo[a]), int(lo[a] + n[a]), device="cuda")) % N] for a in range(3)]
        return (ix[2][:, None, None] * N + ix[1][None, :, None]) * N + ix[0][None, None, :]

    def add(o, at, val):
        if max(at.shape) > N:
            W[o].view(-1).index_put_((at,), val, accumulate=True)
        else:
            W[o].view(-1)[at] += val

    for i, j, lo, n, origin, dbox in pairs:
        at = index(lo, n)
        rho = phi[i].view(-1)[at] * phi[j].view(-1)[at]
        v, C = solve(rho, [float(lo[a] * h - origin[a]) for a in range(3)])
        E -= (1.0 if i == j else 2.0) * h ** 3 * (rho * v).sum()
        if dbox is None:
            add(i, at, v * phi[j].view(-1)[at])
            if i != j:
                add(j, at, v * phi[i].view(-1)[at])
            continue
        for side, (o, q) in enumerate(((i, j), (j, i))[:1 if i == j else 2]):
            bl, bn = dbox[2 * side], dbox[2 * side + 1]
            u = [h * torch.arange(int(bl[a]), int(bl[a] + bn[a]), dtype=torch.float64, device="cuda") - origin[a]
                 for a in range(3)]
            far = solve.multipole(C, *u)
            lo0 = [max(int(lo[a]), int(bl[a])) for a in range(3)]
            hi0 = [min(int(lo[a] + n[a]), int(bl[a] + bn[a])) for a in range(3)]
            big = [slice(lo0[a] - int(bl[a]), hi0[a] - int(bl[a])) for a in (2, 1, 0)]
            small = [slice(lo0[a] - int(lo[a]), hi0[a] - int(lo[a])) for a in (2, 1, 0)]
            far[big[0], big[1], big[2]] = v[small[0], small[1], small[2]]
            at2 = index(bl, bn)
            add(o, at2, far * phi[q].view(-1)[at2])
    return W, E


def _ace_exact(cell, phi, W, psi):
    P, Wm, X = phi.flatten(1), W.flatten(1), psi.double().flatten(1)
    dV = cell.h ** 3
    M = dV * (P @ Wm.T)
    Lm, Li = _inverse_factor(M)
    xi = Li @ Wm
    K = -((dV * (X @ xi.T)) @ xi)
    return {"M": M, "L": Lm, "xi": xi.view_as(W), "Kpsi": K.view(psi.shape), "E": -float((dV * (P @ xi.T)).square().sum())}


def _scdm_exact(phi, W):
    A = phi.double().flatten(1)
    n = A.shape[0]
    res = A.clone()
    taken = torch.zeros(A.shape[1], dtype=torch.bool, device="cuda")
    piv, rd = [], []
    for _ in range(n):
        norms = res.square().sum(0).masked_fill_(taken, -1.0)
        c = int(norms.argmax())
        r = float(norms[c]) ** 0.5
        q = res[:, c] / r
        res.addr_(q, q @ res, alpha=-1.0)
        taken[c] = True
        piv.append(c)
        rd.append(r)
    B = A[:, piv]
    u, _, vt = torch.linalg.svd(B.cpu())
    U = (u @ vt).cuda()
    return {"U": U, "loc": (U.T @ A).view(phi.shape), "piv": np.array(piv, dtype=np.int32), "rdiag": np.array(rd),
            "back": (U @ W.double().flatten(1)).view(phi.shape)}


def _train_exact(case, x, t):
    flat = torch.from_numpy(np.load(WEIGHTS)).float().cuda()
    leaf, w, off = [], {}, 0
    for name, ci, co, relu in sea.NN_LAYERS:
        k = flat[off:off + co * ci * 27]
        if case["weights"] == "bf16":
            k = k.bfloat16()
        off += co * ci * 27
        k, b = k.double().view(co, ci, 27).clone(), flat[off:off + co].double().clone()
        off += co
        k.requires_grad_()
        b.requires_grad_()
        leaf += [k, b]
        w[name] = (k, b, relu)

    def layer(name, inp):
        k, b, relu = w[name]
        D = inp.shape[-1]
        pad = torch.nn.functional.pad(inp, (1,) * 6)
        out = b[None, :, None, None, None].expand(inp.shape[0], -1, D, D, D)
        for tap in range(27):
            z, y, xx = tap // 9, tap // 3 % 3, tap % 3
            win = pad[:, :, z:z + D, y:y + D, xx:xx + D].flatten(2).contiguous()
            out = out + torch.matmul(k[:, :, tap], win).view(out.shape)
        return torch.relu(out) if relu else out

    def up(v):
        for d in (2, 3, 4):
            v = v.repeat_interleave(2, dim=d)
        return v

    pool = torch.nn.functional.avg_pool3d
    X = x.double()[:, None]
    s0 = layer("e0b", layer("e0a", X))
    s1 = layer("e1b", layer("e1a", pool(s0, 2)))
    s2 = layer("e2b", layer("e2a", pool(s1, 2)))
    v = layer("e3b", layer("e3a", pool(s2, 2)))
    for name, skip in (("d2", s2), ("d1", s1), ("d0", s0)):
        v = layer(name + "b", layer(name + "a", torch.cat([up(v), skip], 1)))
    loss = (layer("head", v)[:, 0] - t.double()).square().mean()
    g = torch.autograd.grad(loss, leaf)
    return {"loss": float(loss.detach()), "grad": torch.cat([q.reshape(-1) for q in g])}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("exx", "chain"):
        cell, phi = _orbitals(case, seed, DTYPES[case["phi"]])
        pairs = _eps_pairs(cell, phi, 6) if case.get("rule", "eps") == "eps" else _cube_pairs(cell, case["half"])
        W, E = _exx_exact(cell, phi, pairs)
        return {"W": W, "E": E.reshape(1)}
    if kind == "plan":
        got = [_exx_exact(cell, phi, _cube_pairs(cell, 6.0)) for cell, phi in _plan_cells(case, seed)]
        return {"W": [g[0] for g in got], "E": torch.stack([g[1] for g in got])}
    if kind == "ace":
        return _ace_exact(*_ace_inputs(case, seed))
    if kind == "apply":
        cell, phi, W, psi = _ace_inputs(case, seed)
        xi = _xi(cell, phi, W, DTYPES[case["dtype"]]).double().flatten(1)
        X = psi.double().flatten(1)
        return {"Kpsi": -((cell.h ** 3 * (X @ xi.T)) @ xi).view(psi.shape)}
    if kind == "scdm":
        cell, phi = _delocalized(case, seed)
        return _scdm_exact(phi, (phi * _potential(cell)).to(phi.dtype))
    return _train_exact(case, *_train_inputs(case, seed))
