"""Idle lanes (a spin group's lanes past its electrons, the last wave's missing
walkers) add nothing, whatever they hold.

They sit at the far point (100, 100, 100).  A molecule moved there puts them on
a nucleus, where Slater AOs have infinite derivatives.  The shift is exact (every
coordinate a multiple of 2^-30), so every displacement and with it every result
has to be bit for bit that of the molecule at the origin."""
import numpy as np
import pytest

from paper_2506_09743_amd import synth

pytestmark = pytest.mark.gpu


def _dyadic(x):
    return np.round(np.asarray(x) * 2.0**30) / 2.0**30


@pytest.mark.parametrize("many_body", [False, True], ids=["pade", "many-body"])
@pytest.mark.parametrize("n_up,n_dn", [(3, 3), (3, 1), (4, 0)])
def test_molecule_at_the_far_point(torch_cuda, qmc, n_up, n_dn, many_body):
    torch = torch_cuda
    sysd = synth.make_system("Li2")
    sysd["R"] = _dyadic(sysd["R"])
    if (n_up, n_dn) != (sysd["n_up"], sysd["n_dn"]):
        occ = synth.excitation_dets(n_up, n_dn, sysd["mo_coef"].shape[1], 1)
        sysd = synth._finish(dict(sysd, n_up=n_up, n_dn=n_dn, occ_up=occ[0], occ_dn=occ[1], ci=[1.0]))
    if many_body:
        sysd = synth.with_many_body_jastrow(sysd, synth.MBJ_SEED["Li2"])
    assert sysd["basis"] == "sto"
    X = _dyadic(synth.init_walkers(sysd, 9, 5))
    shift = 100.0 - sysd["R"][0]
    far = dict(sysd, R=sysd["R"] + shift)
    assert np.array_equal(far["R"] - shift, sysd["R"]) and np.array_equal((X + shift) - shift, X)
    out = []
    for d, x in ((sysd, X), (far, X + shift)):
        s = qmc.System(d, device=0)
        t = torch.from_numpy(x).cuda()
        r = {f"eval {p}": s.eval(t, precision=p) for p in ("fp64", "fp32", "fp64_explicit")}
        r.update({f"grad {p}": s.grad(t, precision=p) for p in ("fp64", "fp32")})
        out.append({k: [v.cpu().numpy() for v in vs] for k, vs in r.items()})
        s.close()
    for k, vs in out[0].items():
        for i, (a, b) in enumerate(zip(vs, out[1][k])):
            assert np.isfinite(a).all() and np.array_equal(a, b), (k, i)
