"""qmc_vjp: per-walker weights applied to the qmc_grad outputs.

Against the exactly rounded sum (math.fsum) of the same products.  Each of the
2 W terms enters through one fused multiply-add and the partial sums meet in
additions, so the error is within 2 W u of the sum of the terms' magnitudes
(u = 2^-53), plus u of the products of the reference.  Walker counts lie around
the ranges that the kernel cuts (16 walkers at least, 256 ranges at most).
"""
import math

import numpy as np
import pytest

from paper_2506_09743_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [0, 1, 3, 16, 17, 257, 4096, 4099])
def test_vjp_against_exact_sums(W):
    import torch
    from paper_2506_09743_amd import qmc
    s = qmc.System(synth.make_system("LiH"))
    P, A = s.param_count, s.n_atoms
    g = torch.Generator().manual_seed(W)
    jac = [torch.randn((W, P), generator=g, dtype=torch.float64), torch.randn((W, P), generator=g, dtype=torch.float64),
           torch.randn((W, A, 3), generator=g, dtype=torch.float64),
           torch.randn((W, A, 3), generator=g, dtype=torch.float64)]
    gl, ge = (torch.randn(W, generator=g, dtype=torch.float64) for _ in range(2))
    if W > 2:  # rows of weight zero add nothing, whatever they hold
        gl[1], ge[2] = 0.0, 0.0
        jac[0][1], jac[2][1] = math.nan, math.inf
        jac[1][2], jac[3][2] = math.inf, math.nan
    t, R = s.vjp(gl.cuda(), ge.cuda(), [j.cuda() for j in jac])
    got = torch.cat([t, R.reshape(-1)]).cpu().numpy()
    a = np.concatenate([jac[0].numpy(), jac[2].reshape(W, 3 * A).numpy()], axis=1)
    b = np.concatenate([jac[1].numpy(), jac[3].reshape(W, 3 * A).numpy()], axis=1)
    terms = np.concatenate([np.where(gl.numpy()[:, None] != 0, gl.numpy()[:, None] * np.nan_to_num(a), 0.0),
                            np.where(ge.numpy()[:, None] != 0, ge.numpy()[:, None] * np.nan_to_num(b), 0.0)])
    assert got.shape == (P + 3 * A,)
    for p in range(P + 3 * A):
        bound = (2 * W + 2) * 2.0 ** -53 * np.abs(terms[:, p]).sum()
        assert abs(got[p] - math.fsum(terms[:, p])) <= bound
    if W > 2:  # a non-finite row or weight with a non-zero weight shows
        gl[2] = math.nan
        t, R = s.vjp(gl.cuda(), ge.cuda(), [j.cuda() for j in jac])
        assert torch.isnan(t).all() and torch.isnan(R).all()
    s.close()


def test_backward_forms_agree():
    """One backward pass as it is, recorded for a second derivative, and batched
    over weights: the same gradients (rounding of a sum over 80 walkers)."""
    import torch
    from paper_2506_09743_amd import autograd as ag
    sysd = synth.make_system("H2")
    X = torch.from_numpy(synth.init_walkers(sysd, 40, 3)).cuda()
    wf = ag.Wavefunction(sysd)
    lp, _, el = ag.psi_eloc(wf, X)
    c = torch.linspace(0.5, 1.5, 40, dtype=torch.float64).cuda().requires_grad_()
    plain = torch.autograd.grad((c * lp).mean() + el.mean(), (wf.theta, wf.R), retain_graph=True)
    rec = torch.autograd.grad((c * lp).mean() + el.mean(), (wf.theta, wf.R), retain_graph=True, create_graph=True)
    dl, de, dlR, deR = wf.system().grad(X)
    scale = [(dl.abs().sum(0) * 1.5 + de.abs().sum(0)).cpu(), (dlR.abs().sum(0) * 1.5 + deR.abs().sum(0)).cpu()]
    for p, r, k in zip(plain, rec, scale):
        assert ((p - r.detach()).abs() <= 2 * 82 * 2.0 ** -53 * k / 40).all()
    # the recorded form differentiates to the weights: d (d/dR . 1) / dc_w = sum dlogpsi_dR[w] / W
    (dc,) = torch.autograd.grad(rec[1].sum(), c)
    want = dlR.sum((1, 2)) / 40
    assert ((dc - want).abs() <= 16 * 2.0 ** -53 * dlR.abs().sum((1, 2)) / 40).all()
    g = torch.stack([torch.ones(40, dtype=torch.float64), torch.arange(40, dtype=torch.float64)]).cuda()
    batched = torch.autograd.grad(lp, wf.R, g, retain_graph=True, is_grads_batched=True)[0]
    for i in range(2):
        one = torch.autograd.grad(lp, wf.R, g[i], retain_graph=True)[0]
        k = (g[i].abs()[:, None, None] * dlR.abs()).sum(0).cpu()
        assert ((one - batched[i]).abs() <= 2 * 82 * 2.0 ** -53 * k).all()
    wf.close()
