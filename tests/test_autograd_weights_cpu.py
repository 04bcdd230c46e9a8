"""The weights of a backward pass as the C call gets them: the memory behind the
pointers holds what the tensors mean.  The library's calls are replaced by host
functions that read their pointers, so this runs without a GPU."""
import ctypes as C

import numpy as np
import pytest
import torch

W, P, A = 5, 3, 2


@pytest.fixture
def host_lib(monkeypatch):
    """A System on host memory whose qmc_vjp is a numpy product of what it reads."""
    from paper_2506_09743_amd import qmc

    def read(p, n):
        return np.ctypeslib.as_array((C.c_double * n).from_address(p.value)).copy() if n else np.zeros(0)

    class Lib:
        calls = 0

        def qmc_param_count(self, h):
            return P

        def qmc_vjp_work_bytes(self, h, w):
            return 8

        def qmc_vjp(self, h, gl, ge, dl, de, dlR, deR, w, work, out, stream):
            Lib.calls += 1
            if w and not (gl.value and ge.value):
                return -1
            a = np.c_[read(dl, w * P).reshape(w, P), read(dlR, w * 3 * A).reshape(w, 3 * A)]
            b = np.c_[read(de, w * P).reshape(w, P), read(deR, w * 3 * A).reshape(w, 3 * A)]
            v = np.ascontiguousarray(read(gl, w) @ a + read(ge, w) @ b)
            C.memmove(out.value, v.ctypes.data, v.nbytes)
            return 0

    lib = Lib()
    monkeypatch.setattr(qmc, "lib", lambda: lib)
    monkeypatch.setattr(qmc, "_stream", lambda: C.c_void_p(0))
    monkeypatch.setattr(qmc, "_dev_ptr", lambda t, name, shape=None: C.c_void_p(t.data_ptr()))
    s = qmc.System.__new__(qmc.System)
    s.handle, s.n_atoms, s.n_elec = C.c_void_p(1), A, 2
    g = torch.Generator().manual_seed(3)
    jac = [torch.randn((W, P), generator=g, dtype=torch.float64) for _ in range(2)]
    jac += [torch.randn((W, A, 3), generator=g, dtype=torch.float64) for _ in range(2)]
    s.eval = lambda X: tuple(torch.arange(1.0, X.shape[0] + 1, dtype=torch.float64) for _ in range(3))
    s.grad = lambda X: tuple(j[:X.shape[0]].contiguous() for j in jac)
    yield s, jac, Lib
    s.handle = None  # nothing for the real library to free


class _Wf:
    """What psi_eloc needs of a Wavefunction."""

    def __init__(self, s):
        self.s = s
        self.theta = torch.zeros(P, dtype=torch.float64, requires_grad=True)
        self.R = torch.zeros(A, 3, dtype=torch.float64, requires_grad=True)

    def system(self):
        return self.s


def _weights(n, lazy):
    v = torch.arange(1.0, n + 1, dtype=torch.float64)
    # torch negates these when they are read; their memory holds the opposite sign
    return torch._neg_view(-v) if lazy else v


@pytest.mark.parametrize("n", [1, W])
def test_lazily_negated_weights(host_lib, n):
    s, jac, _ = host_lib
    from paper_2506_09743_amd import autograd as ag
    wf = _Wf(s)
    X = torch.zeros(n, 2, 3, dtype=torch.float64)
    lp, _, el = ag.psi_eloc(wf, X)
    got = {}
    for lazy in (False, True):
        g = _weights(n, lazy)
        assert g.is_neg() == lazy
        got[lazy] = torch.autograd.grad((lp, el), (wf.theta, wf.R), (g, g), retain_graph=True)
    v = _weights(n, False)
    want = (v @ (jac[0] + jac[1])[:n], torch.einsum("w,wak->ak", v, (jac[2] + jac[3])[:n]))
    for a, b, c in zip(got[False], got[True], want):
        assert torch.equal(a, b) and torch.allclose(a, c, rtol=1e-14, atol=1e-14)
    # a loss that reaches it through a conjugate, one walker: stride 1 leaves it lazy
    if n == 1:
        z = torch.complex(torch.zeros(1, dtype=torch.float64), lp).conj().imag.sum()
        (gt,) = torch.autograd.grad(z, wf.theta, retain_graph=True)
        assert torch.allclose(gt, -jac[0][0], rtol=1e-14, atol=0)


@pytest.mark.parametrize("which", [0, 1, 2, 3, 4, 5])
def test_vjp_resolves_every_operand(host_lib, which):
    """System.vjp itself, each of its operands in turn with the lazy bit."""
    s, jac, _ = host_lib
    args = [_weights(W, False), _weights(W, False), *jac]
    want = s.vjp(args[0], args[1], args[2:])
    args[which] = torch._neg_view(-args[which])
    got = s.vjp(args[0], args[1], args[2:])
    assert all(torch.equal(a, b) for a, b in zip(got, want))


class _Held(torch.Tensor):
    """A tensor that keeps its values in another one and has no memory itself."""

    @staticmethod
    def __new__(cls, t):
        return torch.Tensor._make_wrapper_subclass(cls, t.shape, dtype=t.dtype, device=t.device)

    def __init__(self, t):
        self.t = t

    @classmethod
    def __torch_dispatch__(cls, f, types, args=(), kw=None):
        def plain(t):
            return t.t if isinstance(t, _Held) else t
        out = f(*torch.utils._pytree.tree_map(plain, args), **torch.utils._pytree.tree_map(plain, kw or {}))
        return torch.utils._pytree.tree_map(lambda t: _Held(t) if isinstance(t, torch.Tensor) else t, out)


def _values(t):
    return t.t if isinstance(t, _Held) else t


@pytest.mark.parametrize("kind", ["subclass", "zero", "plain", "none"])
def test_weights_without_memory(host_lib, kind):
    """Weights that a kernel cannot read (a wrapper subclass, torch's zero
    tensors without storage) take the torch products, the others the kernel."""
    s, jac, lib = host_lib
    from paper_2506_09743_amd import autograd as ag
    wf = _Wf(s)
    n = 0 if kind == "none" else W
    lp, _, el = ag.psi_eloc(wf, torch.zeros(n, 2, 3, dtype=torch.float64))
    v = _weights(n, False)
    g = {"subclass": _Held(v), "zero": torch._efficientzerotensor((n,), dtype=torch.float64)}.get(kind, v)
    assert kind in ("plain", "none") or g.data_ptr() == 0
    lib.calls = 0
    got = torch.autograd.grad((lp, el), (wf.theta, wf.R), (g, g))
    assert lib.calls == (1 if kind in ("plain", "none") else 0)
    v = torch.zeros(n, dtype=torch.float64) if kind == "zero" else v
    want = (v @ (jac[0] + jac[1])[:n], torch.einsum("w,wak->ak", v, (jac[2] + jac[3])[:n]))
    for a, b in zip(got, want):
        assert torch.allclose(_values(a), b, rtol=1e-14, atol=1e-14)
