"""Timed workloads of the library: what a program that uses it spends its time in.

``listed()`` holds the fixed cases, ``draw(rng)`` draws another of the same
ranges, ``prepare`` makes a case's inputs and system handle on the GPU,
``run`` is one pass through the public entry points and ``work`` counts the
bytes and operations the pass cannot do without.  ``exact`` evaluates the
same quantities from their definitions with plain torch operations in FP64.

Kinds of case
  block     Metropolis block: ``steps`` all-electron moves of ``walkers``
            walkers with log|Psi| and E_L at each (sampling, serving chunks)
  eval      log|Psi|, sign and E_L of given walkers
  grad      per-walker derivatives of log|Psi| and E_L (parameters, nuclei)
  train     one optimiser step's forward and backward through autograd

The molecules and their sizes are the package's own (``synth``): H2, LiH, Li2
and CO.  ``sd`` takes the SD(sd, sd) expansion (4 to 361 determinants, the
reference's weight 1, the others' 0.05): with a leading reference few walkers
come near a node of the reference determinant, where rounding is amplified,
so outputs can be compared to many digits.  ``many_body`` adds the e-n and
e-e-n Jastrow terms and ``omega`` the inverse backflow.
"""
import math

import numpy as np
import torch

from paper_2506_09743_amd import qmc, synth
from paper_2506_09743_amd.autograd import Wavefunction, pack_theta, psi_eloc

SIGMA = synth.CONFIG_SIGMA
BURN = 20  # sampling steps behind the walkers of an evaluation or derivative call
DEVICE = "cuda"


def _case(kind, molecule, walkers, steps=0, precision="fp64", sd=0, many_body=False, omega=0.0, bond=1.0):
    return dict(kind=kind, molecule=molecule, walkers=walkers, steps=steps, precision=precision, sd=sd,
                many_body=many_body, omega=omega, bond=bond)


def listed():
    def named(name, c):
        c["name"] = name
        return c

    return [
        # the smallest sampling run: launches and latency count, not throughput
        named("h2_block_1k", _case("block", "H2", 1024, 200)),
        # a request of the serving mix, one 50-step chunk of a small molecule
        named("lih_block_16k", _case("block", "LiH", 16384, 50, sd=2)),
        # the same in the mixed form that half of the mix asks for, ragged count
        named("li2_block_fp32_11k", _case("block", "Li2", 11003, 50, precision="fp32", sd=2, bond=1.7)),
        # a mid-sized request of the largest molecule, 118 determinants: a wave or so per SIMD
        named("co_block_5k", _case("block", "CO", 5003, 50, sd=6, bond=1.2)),
        # production sampling: the headline walker count, and its mixed form
        named("co_block_64k", _case("block", "CO", 65536, 10, sd=4)),
        named("co_block_fp32_64k", _case("block", "CO", 65536, 10, precision="fp32", sd=4)),
        # sampling with the many-body Jastrow factor
        named("co_block_manybody_16k", _case("block", "CO", 16384, 10, sd=6, many_body=True)),
        # sampling with the inverse backflow
        named("co_block_backflow_8k", _case("block", "CO", 8192, 3, sd=4, omega=0.1)),
        # energies of a given walker set with 361 determinants (1000 walkers: latency)
        named("co_eval_sd8_1k", _case("eval", "CO", 1000, sd=8)),
        # energies of a given walker set in the matrix-core form
        named("co_eval_bf16_20k", _case("eval", "CO", 20001, precision="bf16", sd=4)),
        # every per-walker derivative: what the optimiser's statistics and the forces need
        named("li2_grad_32k", _case("grad", "Li2", 32768, sd=2)),
        # one optimiser step (E and dE/d(theta, R)) of the largest molecule with every parameter kind
        named("co_train_manybody_4k", _case("train", "CO", 4099, sd=2, many_body=True)),
    ]


def draw(rng):
    """One more case: walkers and steps over the listed ranges, never more
    work than the largest listed case."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = max(work(c)["flops"] for c in listed())
    while True:
        molecule = rng.choice(["H2", "LiH", "Li2", "CO"])
        kind = rng.choice(["block", "block", "block", "eval", "grad", "train"])
        c = _case(kind, molecule, log_int(1000, 65536), bond=round(rng.uniform(0.6, 3.0), 3))
        if kind == "block":
            c["steps"] = rng.choice([3, 10, 25, 50])
        if kind in ("block", "eval"):
            option = rng.choice(["", "", "fp32", "fp32", "bf16", "many_body", "backflow"])
            if option in ("fp32", "bf16"):
                c["precision"] = option
            elif option == "many_body":
                c["many_body"] = True
            elif option == "backflow":
                c["omega"] = round(rng.uniform(0.05, 0.3), 3)
                c["walkers"] = log_int(1000, 8192)
                c["steps"] = min(c["steps"], 3)
        else:
            c["walkers"] = log_int(1000, 32768 if kind == "grad" else 8192)
            c["many_body"] = rng.random() < 0.4
        if molecule != "H2":
            small = c["walkers"] * (c["steps"] or BURN) < 100000
            c["sd"] = rng.choice([2, 4, 6, 8] if molecule == "CO" and small and kind in ("block", "eval")
                                 else [2, 4] if molecule == "CO" and kind == "block" else [2])
        if work(c)["flops"] <= most:
            return c


def _system(c):
    sysd = synth.make_system(c["molecule"], bond_scale=c["bond"])
    if c["sd"]:
        sysd = synth.with_sd_expansion(sysd, c["sd"], 5)
    if c["many_body"]:
        sysd = synth.with_many_body_jastrow(sysd, synth.MBJ_SEED[c["molecule"]])
    if c["omega"]:
        sysd["bf_omega"] = c["omega"]
    return sysd


def _walkers(sysd, c, seed):
    return synth.init_walkers_device(sysd, c["walkers"], seed, DEVICE)


def prepare(c, seed):
    sysd = _system(c)
    X = _walkers(sysd, c, seed)
    state = dict(case=c, X=X, step=0, seed=int(seed))
    if c["kind"] == "train":
        state["wf"] = Wavefunction(sysd, 0)
        system = state["wf"].system()
    else:
        system = state["sys"] = qmc.System(sysd, 0)
    if c["kind"] == "block":
        state["psi"] = system.eval(X, precision=c["precision"])
        state["acc"] = torch.zeros((c["walkers"], qmc.ACC_COLS), dtype=torch.float64, device=X.device)
    else:
        # energies and derivatives are taken at sampled walkers
        system.metropolis(X, *system.eval(X), BURN, SIGMA, state["seed"])
    return state


def run(s):
    c, X = s["case"], s["X"]
    if c["kind"] == "block":
        s["sys"].metropolis(X, *s["psi"], c["steps"], SIGMA, s["seed"], step0=s["step"], acc=s["acc"],
                            precision=c["precision"])
        s["step"] += c["steps"]
        return dict(X=X, psi=s["psi"], acc=s["acc"])
    if c["kind"] == "eval":
        return dict(psi=s["sys"].eval(X, precision=c["precision"]))
    if c["kind"] == "grad":
        return dict(grad=s["sys"].grad(X, precision=c["precision"]))
    wf = s["wf"]
    wf.theta.grad = wf.R.grad = None
    lp, _, el = psi_eloc(wf, X)
    energy = el.detach().mean()
    loss = el.mean() + 2.0 * ((el.detach() - energy) * lp).mean()
    loss.backward()
    return dict(lp=lp.detach(), el=el.detach(), energy=energy, theta=wf.theta.grad, R=wf.R.grad)


def work(c):
    """Operations (a multiply-add is two, every other one) and HBM bytes."""
    sysd = _system(c)
    nu, nd = int(sysd["n_up"]), int(sysd["n_dn"])
    ne, na, nmo, nao = nu + nd, len(sysd["Z"]), sysd["mo_coef"].shape[1], synth.n_ao(sysd)
    ndet, nprim, nsh = len(sysd["ci"]), sysd["prim_exp"].size, len(sysd["shell_l"])
    pairs = ne * (ne - 1) // 2
    n_par = pack_theta(sysd).size
    rank = [(sysd[k] != sysd[k][0]).sum(axis=1) for k in ("occ_up", "occ_dn")]
    cofactors = sum(int((r == 1).sum()) + 4 * int((r == 2).sum()) for r in rank)
    ao = ne * (10 * nsh + (17 if sysd["basis"] == "sto" else 13) * nprim + 10 * nao)
    dets = sum(2 * n * n * nmo + n * (4 * n * (nmo - n) + 8 * nmo) for n in (nu, nd)) + 8 * ndet + 6 * cofactors
    jastrow = 25 * pairs + 9 * ne * na
    if c["many_body"]:
        jastrow += 20 * ne * na + na * pairs * 65 * len(sysd["jas_een"]) + 12 * ne * na
    # values and, by the adjoint vector, one weight per AO: two contractions
    flops = ao + 4 * ne * nao * nmo + dets + jastrow + 15 * ne
    if c["omega"]:
        ncfg = [len({tuple(r) for r in sysd[k].tolist()}) for k in ("occ_up", "occ_dn")]
        blocks = nu * (nu + 1) // 2 + nd * (nd + 1) // 2 + nu * nd
        flops = 2 * ao + 10 * ne * nao * nmo + jastrow + 47 * ne * (ne - 1) + 54 * blocks * ne
        for n, k, o in ((nu, ncfg[0], nd), (nd, ncfg[1], nu)):
            flops += 2 * n * n * nmo + 16 * n * n * nmo + k * (12 * n * n + 24 * n * (n + 1) + 12 * n * o)
        flops += ndet * (4 + 6 * ne)
    W, doubles = c["walkers"], 3 * ne + 3
    if c["kind"] == "block":
        # the state and the accumulators once each way
        return dict(bytes=8 * W * 2 * (3 * ne + 7), flops=W * c["steps"] * (flops + 20 * ne + 6))
    if c["kind"] in ("grad", "train"):
        # forward, the direction B and its contraction, the forward-mode
        # determinants, the exponent and nuclear passes, the MO outer products
        flops = 2 * flops + 2 * ne * nao * nmo + dets + 3 * ao + 6 * ne * nao * nmo
        # E and its derivatives alone leave the training step; grad writes every walker's
        doubles = 3 * ne + (2 * (n_par + 3 * na) if c["kind"] == "grad" else 2)
    return dict(bytes=8 * W * doubles, flops=W * flops)


# ---- the same quantities from their definitions, plain torch in FP64 -----------------

class _Model:
    """log|Psi| and E_L of walkers X [W, N_e, 3] from a system's tables.
    ``theta`` (the optimiser's layout) and ``R`` may carry a leading walker
    axis, so that one backward pass gives every walker's own derivatives."""

    def __init__(self, sysd, theta=None, R=None):
        f = lambda v: torch.as_tensor(np.asarray(v, dtype=np.float64), device=DEVICE)  # noqa: E731
        self.d = d = sysd
        self.nu, self.nd = int(d["n_up"]), int(d["n_dn"])
        self.ne = self.nu + self.nd
        self.Z = f(d["Z"])
        self.R = (f(d["R"]) if R is None else R)
        self.R = self.R if self.R.dim() == 3 else self.R[None]
        th = f(pack_theta(d)) if theta is None else theta
        th = th if th.dim() == 2 else th[None]
        nao, nmo = d["mo_coef"].shape
        sizes = [d["prim_exp"].size, nao * nmo, 1]
        self.en = d.get("jas_en") is not None
        self.een = d.get("jas_een") is not None and len(d["jas_een"]) > 0
        sizes += [3 * len(d["Z"])] if self.en else []
        sizes += [7 * len(d["jas_een"])] if self.een else []
        part = list(torch.split(th, sizes, dim=1))
        self.exps, self.C, self.b = part[0], part[1].reshape(-1, nao, nmo), part[2]
        if self.en:
            self.w_en = part[3].reshape(th.shape[0], -1, 3)
        if self.een:
            self.t_een = part[-1].reshape(th.shape[0], -1, 7)
        self.coef, self.ci = f(d["prim_coef"]), f(d["ci"])

    def orbitals(self, q, want):
        """MO values of the electrons at q and, wanted, gradient and Laplacian."""
        d, sto = self.d, self.d["basis"] == "sto"
        chi, grad, lap = [], [], []
        p = 0
        for a, l, kn, n in zip(*(d[k].tolist() for k in ("shell_atom", "shell_l", "shell_kn", "shell_nprim"))):
            v = q - self.R[:, None, a]
            r2 = (v * v).sum(-1)
            r = r2.sqrt()
            e = self.exps[:, None, p:p + n]
            c = self.coef[p:p + n]
            if d["normalize"]:
                if sto:
                    k = l + kn + 1
                    c = c * (2 * e) ** (k + 0.5) * math.sqrt(math.prod(range(2 * l + 1, 0, -2))
                                                             / math.factorial(2 * k) / (4 * math.pi))
                else:
                    c = c * (2 * e / math.pi) ** 0.75 * (4 * e) ** (0.5 * l)
            p += n
            if sto:
                f = c * (r ** kn)[..., None] * torch.exp(-e * r[..., None])
                g = kn / r[..., None] - e
                f1, f2 = f * g, f * (g * g - kn / r2[..., None])
            else:
                f = c * torch.exp(-e * r2[..., None])
                f1, f2 = -2 * e * r[..., None] * f, f * (4 * e * e * r2[..., None] - 2 * e)
            f, f1, f2 = f.sum(-1), f1.sum(-1), f2.sum(-1)
            for i in range(l, -1, -1):
                for j in range(l - i, -1, -1):
                    pw = (i, j, l - i - j)
                    ang = 1.0
                    for m in pw:
                        ang /= math.sqrt(math.prod(range(2 * m - 1, 0, -2))) if d["normalize"] else 1.0
                    mono = [v[..., x] ** pw[x] for x in range(3)]
                    P = ang * mono[0] * mono[1] * mono[2]
                    chi.append(P * f)
                    if not want:
                        continue
                    dP = []
                    lapP = 0.0
                    for x in range(3):
                        rest = ang * mono[(x + 1) % 3] * mono[(x + 2) % 3]
                        dP.append(pw[x] * v[..., x] ** max(pw[x] - 1, 0) * rest)
                        if pw[x] > 1:
                            lapP = lapP + pw[x] * (pw[x] - 1) * v[..., x] ** (pw[x] - 2) * rest
                    grad.append(torch.stack([dP[x] * f + P * f1 * v[..., x] / r for x in range(3)], -1))
                    lap.append(lapP * f + P * (f2 + (2 * l + 2) * f1 / r))
        C = self.C
        phi = torch.stack(chi, -1) @ C
        if not want:
            return phi
        g = torch.stack(grad, -2)  # [W, e, ao, 3]
        return phi, torch.stack([g[..., x] @ C for x in range(3)], -1), torch.stack(lap, -1) @ C

    def ratio(self, T, occ):
        """det(A_n) / det(A_0) of one spin for every determinant: at most two
        of its slots hold another orbital than the reference's."""
        n = occ.shape[1]
        if n == 0:
            return torch.ones((T.shape[0], occ.shape[0]), dtype=T.dtype, device=T.device)
        k = min(2, n)
        slots = np.argsort(occ == occ[0], axis=1, kind="stable")[:, :k]
        orb = np.take_along_axis(occ, slots, axis=1)
        slots, orb = (torch.as_tensor(v.astype(np.int64), device=DEVICE) for v in (slots, orb))
        m = lambda i, j: T[:, slots[:, i], orb[:, j]]  # noqa: E731
        return m(0, 0) if k == 1 else m(0, 0) * m(1, 1) - m(0, 1) * m(1, 0)

    def log_sigma(self, phi):
        """log|Sigma| and its sign, Sigma the CI sum over the determinants."""
        log, sign, rho = 0.0, 1.0, 1.0
        for n, rows, occ in ((self.nu, phi[:, :self.nu], self.d["occ_up"]), (self.nd, phi[:, self.nu:], self.d["occ_dn"])):
            if n == 0:
                continue
            A = rows[..., torch.as_tensor(occ[0].astype(np.int64), device=DEVICE)]
            s, lg = torch.linalg.slogdet(A)
            log, sign = log + lg, sign * s
            rho = rho * self.ratio(torch.linalg.inv(A) @ rows, occ)
        S = (self.ci * rho).sum(-1)
        return log + S.abs().log(), sign * S.sign()

    def jastrow(self, X):
        """J, its gradient and Laplacian per electron, and the Coulomb energy."""
        ne = self.ne
        up = torch.arange(ne, device=DEVICE) < self.nu
        eye = torch.eye(ne, dtype=torch.float64, device=DEVICE)
        u = X[:, :, None] - X[:, None]
        r = ((u * u).sum(-1) + eye).sqrt()
        off = 1.0 - eye
        a = torch.where(up[:, None] == up, float(self.d["jas_a_par"]), float(self.d["jas_a_anti"])) * off
        b = self.b[:, None]
        den = 1 + b * r
        k1, k2 = a / den ** 2, -2 * a * b / den ** 3
        J = 0.5 * (a * r / den).sum((1, 2))
        w = u / r[..., None]
        g = (k1[..., None] * w).sum(2)
        lap = (k2 + 2 * k1 / r).sum(2)
        v = X[:, :, None] - self.R[:, None]
        s = (v * v).sum(-1).sqrt()
        V = 0.5 * (off / r).sum((1, 2)) - (self.Z / s).sum((1, 2))
        Rn = self.R[:, :, None] - self.R[:, None]
        for i in range(len(self.Z)):
            for j in range(i):
                V = V + self.Z[i] * self.Z[j] / (Rn[:, i, j] ** 2).sum(-1).sqrt()
        t = v / s[..., None]
        if self.en:
            w0, w1, w2 = (self.w_en[:, None, :, k] for k in range(3))
            D = 1 + w2 * s
            K = (w0 * s + w1 * s * s) / D
            K1 = (w0 + 2 * w1 * s - K * w2) / D
            K2 = (2 * w1 - 2 * K1 * w2) / D
            J, g, lap = J + K.sum((1, 2)), g + (K1[..., None] * t).sum(2), lap + (K2 + 2 * K1 / s).sum(2)
        if self.een:
            lower = (torch.arange(ne, device=DEVICE)[:, None] > torch.arange(ne, device=DEVICE)).double()

            def kernel(x, A, B):
                D = 1 + B * x
                return A * x / D, A / D ** 2, -2 * A * B / D ** 3

            for m in range(self.t_een.shape[1]):
                c, a1, b1, a2, b2, a3, b3 = (self.t_een[:, None, None, m, k] for k in range(7))
                F1, F2, F3 = kernel(s, a1, b1), kernel(s, a2, b2), kernel(r, a3, b3)
                for n in range(len(self.Z)):
                    uw = torch.einsum("wix,wijx->wij", t[:, :, n], w)
                    for own, oth, pick in ((F1, F2, lower), (F2, F1, lower.T)):
                        o, o1, o2 = (k[:, :, None, n] for k in own)
                        P = c * oth[0][:, None, :, n] * pick
                        if pick is lower:
                            J = J + (P * o * F3[0]).sum((1, 2))
                        g = g + (P * o1 * F3[0]).sum(2)[..., None] * t[:, :, n] + ((P * o * F3[1])[..., None] * w).sum(2)
                        lap = lap + (P * ((o2 + 2 * o1 / s[:, :, None, n]) * F3[0] + 2 * o1 * F3[1] * uw
                                          + o * (F3[2] + 2 * F3[1] / r))).sum(2)
        return J, g, lap, V

    def psi_eloc(self, X, graph=False):
        """log|Psi|, sign and E_L."""
        if self.d.get("bf_omega"):
            return self.psi_eloc_backflow(X)
        with torch.enable_grad():
            phi, dphi, lphi = self.orbitals(X, True)
            leaf = phi if graph else phi.detach().requires_grad_()
            ls, sign = self.log_sigma(leaf)
            adj, = torch.autograd.grad(ls.sum(), leaf, create_graph=graph)
        J, gJ, lapJ, V = self.jastrow(X)
        gS = (adj[..., None] * dphi).sum(2)
        kin = -0.5 * ((adj * lphi).sum((1, 2)) + lapJ.sum(1) + (gJ * gJ).sum((1, 2)) + 2 * (gJ * gS).sum((1, 2)))
        out = J + ls, sign, kin + V
        return out if graph else tuple(t.detach() for t in out)

    def psi_eloc_backflow(self, X):
        """Orbitals at the transformed positions; the kinetic energy from
        second derivatives of log|Psi| along every coordinate."""
        with torch.enable_grad():
            X = X.detach().requires_grad_()
            u = X[:, :, None] - X[:, None]
            eye = torch.eye(self.ne, dtype=torch.float64, device=DEVICE)
            r = ((u * u).sum(-1) + eye).sqrt()
            q = X + ((float(self.d["bf_omega"]) / r)[..., None] * u).sum(2)
            ls, sign = self.log_sigma(self.orbitals(q, False))
            J, gJ, lapJ, V = self.jastrow(X)
            g, = torch.autograd.grad(ls.sum(), X, create_graph=True)
            flat = g.reshape(X.shape[0], -1)
            lap = 0.0
            for k in range(flat.shape[1]):
                h, = torch.autograd.grad(flat[:, k].sum(), X, retain_graph=True)
                lap = lap + h.reshape(X.shape[0], -1)[:, k]
        kin = -0.5 * (lap + (g * g).sum((1, 2)) + lapJ.sum(1) + (gJ * gJ).sum((1, 2)) + 2 * (gJ * g).sum((1, 2)))
        return tuple(t.detach() for t in (J + ls, sign, kin + V))


def _chunks(fn, X, size):
    parts = [fn(X[i:i + size]) for i in range(0, X.shape[0], size)]
    return tuple(torch.cat(p) for p in zip(*parts))


def _philox(c, key):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    mask = 0xFFFFFFFF
    k0, k1 = key & mask, (key >> 32) & mask
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & mask) ^ c[1] ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c[3] ^ k1, p0 & mask]
    return c


def _moves(seed, step, W, ne):
    """The step's normals [W, N_e, 3] and acceptance uniforms [W]."""
    w = torch.arange(W, dtype=torch.int64, device=DEVICE)[:, None]
    e = torch.arange(ne + 1, dtype=torch.int64, device=DEVICE)[None]
    zero = torch.zeros_like(w + e)
    c = _philox([zero + w, zero + (step & 0xFFFFFFFF), zero + (step >> 32), zero + e], seed)
    u = [(v[:, :ne].double() + 0.5) / 4294967296.0 for v in c]
    r0, r1 = (-2 * u[0].log()).sqrt(), (-2 * u[2].log()).sqrt()
    a, b = 2 * math.pi * u[1], 2 * math.pi * u[3]
    z = torch.stack([r0 * a.cos(), r0 * a.sin(), r1 * b.cos()], -1)
    bits = ((c[0][:, ne] << 21) | (c[1][:, ne] >> 11))
    return z, bits.double() / 9007199254740992.0


def _sample(m, X, steps, seed, size):
    """The Metropolis chain of walkers X: end state and accumulators."""
    psi = _chunks(m.psi_eloc, X, size)
    acc = torch.zeros((X.shape[0], qmc.ACC_COLS), dtype=torch.float64, device=X.device)
    for t in range(steps):
        z, u = _moves(int(seed), t, X.shape[0], m.ne)
        Y = X + SIGMA * z
        new = _chunks(m.psi_eloc, Y, size)
        take = u < torch.exp(2 * (new[0] - psi[0]))
        X = torch.where(take[:, None, None], Y, X)
        psi = tuple(torch.where(take, n, o) for n, o in zip(new, psi))
        el = psi[2]
        acc += torch.stack([el, el * el, take.double(), torch.zeros_like(el)], 1)
    return X, psi, acc


def exact(c, seed):
    sysd = _system(c)
    W, block = c["walkers"], c["kind"] == "block"
    m, size = _Model(sysd), 4096 if c["many_body"] else 8192
    steps = c["steps"] if block else BURN
    if c["omega"] and (steps + 1) * W > 40000 or c["many_body"] and (steps + 1) * W > 400000:
        return None
    X, psi, acc = _sample(m, _walkers(sysd, c, seed), steps, seed, size)
    if block:
        return dict(X=X, psi=psi, acc=acc)
    if c["kind"] == "eval":
        return dict(psi=psi)

    def derivatives(x):
        """Every walker's own derivatives: the parameters with a walker axis."""
        theta = torch.as_tensor(pack_theta(sysd), device=DEVICE).expand(len(x), -1).clone().requires_grad_()
        R = torch.as_tensor(np.asarray(sysd["R"]), device=DEVICE).expand(len(x), -1, -1).clone().requires_grad_()
        lp, _, el = _Model(sysd, theta, R).psi_eloc(x, graph=True)
        dl = torch.autograd.grad(lp.sum(), (theta, R), retain_graph=True)
        de = torch.autograd.grad(el.sum(), (theta, R))
        return lp.detach(), el.detach(), dl[0], de[0], dl[1], de[1]

    lp, el, dl, de, dlR, deR = _chunks(derivatives, X, 2048)
    if c["kind"] == "grad":
        return dict(grad=(dl, de, dlR, deR))
    energy = el.mean()
    weight = 2 * (el - energy) / W
    total = lambda de_, dl_: (de_.mean(0) + torch.tensordot(weight, dl_, 1)).cpu()  # noqa: E731
    return dict(lp=lp, el=el, energy=energy, theta=total(de, dl), R=total(deR, dlR))
