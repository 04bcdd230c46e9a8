"""The e-e-n Jastrow terms on the paths the evaluation and the adjoint choose
between: symmetric terms (one role) and asymmetric ones (two), one to three
nuclei (they are taken two at a time), no electron pair, and terms whose
coefficients vanish (every parameter's derivative stays finite), against the
FP64 oracle and its central differences."""
import numpy as np
import pytest

from paper_2506_09743_amd import synth
from parity_helpers import _compare

pytestmark = pytest.mark.gpu


def _system(n_atoms, n_up, n_dn, kinds, seed):
    rng = np.random.default_rng(seed)
    R = np.array([[0.0, 0.0, -1.1], [0.2, 0.1, 1.0], [1.3, -0.4, 0.1]])[:n_atoms]
    l = [0, 1] * n_atoms
    nao = sum(synth.n_cart(v) for v in l)
    occ_up, occ_dn = synth.excitation_dets(n_up, n_dn, nao, 1)
    d = synth._finish(dict(
        name="roles", Z=[2.0, 3.0, 1.0][:n_atoms], R=R, n_up=n_up, n_dn=n_dn, basis="sto",
        shell_atom=[i // 2 for i in range(2 * n_atoms)], shell_l=l, shell_kn=[0] * len(l), shell_nprim=[1] * len(l),
        prim_exp=rng.uniform(0.6, 1.8, len(l)), prim_coef=np.ones(len(l)), mo_coef=synth.orthogonal(nao, rng),
        occ_up=occ_up, occ_dn=occ_dn, ci=[1.0], jas_b=0.8))
    d["jas_en"] = np.c_[rng.uniform(-0.3, 0.3, n_atoms), rng.uniform(-0.1, 0, n_atoms), rng.uniform(0.5, 2, n_atoms)]
    een = np.c_[rng.normal(0, 0.2, len(kinds)), rng.uniform(0.4, 1.2, (len(kinds), 6))]
    for m, k in enumerate(kinds):
        if k == "sym":
            een[m, 3:5] = een[m, 1:3]
        elif k == "zero":
            een[m, [0, 1, 3, 5][m % 4]] = 0.0
        elif k == "half":  # equal a, different b: two roles
            een[m, 3] = een[m, 1]
    d["jas_een"] = een
    return d


CASES = [(1, 2, 1, ["sym", "asym"], 1), (2, 2, 2, ["half", "sym", "zero"], 2), (3, 3, 2, ["asym", "sym"], 3),
         (3, 1, 0, ["sym", "asym"], 4), (2, 3, 3, ["zero", "zero", "zero", "zero"], 5)]


@pytest.mark.parametrize("n_atoms,n_up,n_dn,kinds,seed", CASES)
def test_een_roles(torch_cuda, qmc, oracle_mod, n_atoms, n_up, n_dn, kinds, seed):
    torch = torch_cuda
    d = _system(n_atoms, n_up, n_dn, kinds, seed)
    X = synth.init_walkers(d, 37, 90 + seed)
    s = qmc.System(d, device=0)
    print(f"e-e-n roles {n_atoms} nuclei ({n_up},{n_dn}) {kinds}", flush=True)
    tX = torch.from_numpy(X).cuda()
    lp, sg, el = [t.cpu().numpy() for t in s.eval(tX)]
    _compare(oracle_mod.OracleSystem(d), d, X, lp, sg, el, "e-e-n roles")
    dl, de, dlR, deR = [t.cpu().numpy() for t in s.grad(tX)]
    assert all(np.isfinite(v).all() for v in (dl, de, dlR, deR))
    first = d["prim_exp"].size + d["mo_coef"].size

    def central(key, at, h):
        out = []
        for sign in (1, -1):
            q = dict(d)
            v = np.array(q[key], dtype=np.float64)
            v[at] += sign * h
            q[key] = float(v) if v.ndim == 0 else v
            out.append(oracle_mod.OracleSystem(q).eval(X))
        return [(out[0][k] - out[1][k]) / (2 * h) for k in (0, 2)]

    def differences(key, at):
        """Central differences of the oracle at h and h / 2, extrapolated: an
        electron 0.01 bohr from a moved nucleus has h^2 d^3E/dR^3 = 0.1 Ha/bohr
        at h = 1e-5, which only the h^4 rule resolves."""
        return [(4 * f - c) / 3 for f, c in zip(central(key, at, 5e-6), central(key, at, 1e-5))]

    checks = [("jas_b", (), first)]
    checks += [("jas_en", (a, k), first + 1 + 3 * a + k) for a in range(n_atoms) for k in range(3)]
    checks += [("jas_een", (m, k), first + 1 + 3 * n_atoms + 7 * m + k) for m in range(len(kinds)) for k in range(7)
               if not (k in (2, 4, 6) and d["jas_een"][m, k] < 1e-4)]
    for key, at, col in checks:
        fl, fe = differences(key, at)
        for got, want in ((dl[:, col], fl), (de[:, col], fe)):
            assert np.max(np.abs(got - want)) <= 2e-6 * max(1.0, np.abs(want).max(), np.abs(el).max()), (key, at)
    for a in range(n_atoms):
        for k in range(3):
            fl, fe = differences("R", (a, k))
            for got, want in ((dlR[:, a, k], fl), (deR[:, a, k], fe)):
                assert np.max(np.abs(got - want)) <= 2e-6 * max(1.0, np.abs(want).max(), np.abs(el).max()), ("R", a, k)
    s.close()
