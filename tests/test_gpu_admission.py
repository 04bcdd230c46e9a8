"""Systems by the number of nuclei with eight e-e-n terms: the last that a form
takes and the first that it refuses for want of LDS.  The limits are the
documented formulas, not the present kernels' tables, so they hold from build to
build: two lanes a walker, 32 walkers a wave, 160 KiB = 640 doubles a walker.
Tables of 21 doubles per lane and nucleus and 6 of positions: 42 n + 6; for the
derivatives twice the tables and 6 sums per nucleus: 90 n + 6."""
import numpy as np
import pytest

from paper_2506_09743_amd import synth

pytestmark = pytest.mark.gpu


def _chain(n, omega=0.0):
    rng = np.random.default_rng(n)
    occ_up, occ_dn = synth.excitation_dets(1, 1, 2, 1)
    d = synth._finish(dict(
        name="chain", Z=np.ones(n), R=np.c_[np.zeros(n), np.zeros(n), 1.6 * np.arange(n)], n_up=1, n_dn=1, basis="sto",
        shell_atom=np.arange(n), shell_l=[0] * n, shell_kn=[0] * n, shell_nprim=[1] * n, prim_exp=[1.2] * n,
        prim_coef=[1.0] * n, mo_coef=synth.orthogonal(n, rng)[:, :2], occ_up=occ_up, occ_dn=occ_dn, ci=[1.0],
        jas_b=1.0))
    d["jas_een"] = np.c_[rng.normal(0, 0.01, 8), rng.uniform(0.4, 1.2, (8, 6))]
    d["bf_omega"] = omega
    return d


@pytest.mark.parametrize("what,last", [("fp64_explicit", 15), ("backflow fp64", 15), ("backflow fp64_explicit", 15),
                                       ("grad", 7)])
def test_een_nuclei_limit(torch_cuda, qmc, what, last):
    torch = torch_cuda
    for n in (last, last + 1):
        sysd = _chain(n, 0.1 if "backflow" in what else 0.0)
        X = torch.from_numpy(synth.init_walkers(sysd, 5, 1)).cuda()
        s = qmc.System(sysd, device=0)
        print(f"{what} {n} nuclei", flush=True)

        def call():
            return s.grad(X) if what == "grad" else s.eval(X, what.split()[-1])
        if n > last:
            with pytest.raises(qmc.QmcError) as e:
                call()
            assert e.value.status == qmc.QMC_EUNSUPPORTED
        else:
            assert all(torch.isfinite(t).all() for t in call())
        s.close()
