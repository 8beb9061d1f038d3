"""Outputs in the memory of the inputs, on the grid engine: a launch of one segment stores its
outputs itself, so with shared memory the finalize launch has to store them instead.  Against
the same call with outputs of their own: the sums are the same, bitwise but for the (hi, lo)
FP32 pair that holds a compensated segment sum on its way to the finalize (2^-47 of it)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import _lib, api, ics  # noqa: E402

DEV = "cuda"
EPS = 0.02
SHAPE = {"ipl": 1, "jtile": 128, "nseg": 1, "jlanes": 1}  # one segment at any size


def state(n):
    pos, vel, mass = ics.plummer(n, seed=3)
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    return f(pos.T), f(vel.T), f(mass.astype(np.float32))


def same(a, b, precision):
    if precision == "comp":
        assert float((a - b).abs().max()) <= 2.0 ** -47 * float(b.abs().max())
    else:
        assert torch.equal(a, b)


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("n", [1, 65, 700, 2300])
def test_fp64_outputs_over_fp64_inputs(precision, n):
    x, v, m = state(n)
    for kw in ({"centre": "tile"}, {"centre": "tile", **SHAPE}, {"centre": "system", **SHAPE},
               {"centre": "none"}):
        acc, pot = api.force_f64(x, m, EPS, precision=precision, **kw)
        buf, p = x.clone(), torch.empty_like(pot)
        api.force_f64(buf, m, EPS, precision=precision, out=(buf, p), **kw)
        same(buf, acc, precision)
        same(p, pot, precision)

        ref = api.force_jerk(x, v, m, EPS, precision=precision, **kw)
        a, j = x.clone(), v.clone()
        api.force_jerk(a, j, m, EPS, precision=precision, out=(a, j, p), **kw)
        for got, want in zip((a, j, p), ref):
            same(got, want, precision)

        g = torch.randn((3, n), dtype=torch.float64, device=DEV)
        gp = torch.randn(n, dtype=torch.float64, device=DEV)
        opts = api.make_opts(precision=precision, **kw)

        def vjp(pos, ga, gpot, grad, grad_m):
            _lib.nbody_force_vjp_f64(n, pos.data_ptr(), m.data_ptr(), EPS, ga.data_ptr(),
                                     gpot.data_ptr(), grad.data_ptr(), grad_m.data_ptr(), opts,
                                     api.stream_ptr())
            return grad, grad_m

        want = vjp(x, g, gp, torch.empty_like(g), torch.empty_like(gp))
        a, b = g.clone(), gp.clone()
        for got, w in zip(vjp(x, a, b, a, b), want):
            same(got, w, precision)
        a = x.clone()
        for got, w in zip(vjp(a, g, gp, a, torch.empty_like(gp)), want):
            same(got, w, precision)


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("ni,n", [(64, 300), (700, 700), (200, 2300)])
def test_fp64_outputs_over_fp32_inputs(precision, ni, n):
    x, v, m = (t.float() for t in state(n))
    xi, vi = x[:, :ni].contiguous(), v[:, :ni].contiguous()

    def over(t):  # a copy of t in the first half of the memory of an output
        out = torch.empty(t.shape, dtype=torch.float64, device=DEV)
        t32 = out.view(-1).view(torch.float32)[: t.numel()].view(t.shape)
        t32.copy_(t)
        return t32, out

    kw = dict(precision=precision, with_pot=False)
    want = api.force(x, m, EPS, **kw, **SHAPE)[0]
    p, a = over(x)
    api.force(p, m, EPS, out=(a, None), **kw, **SHAPE)
    same(a, want, precision)
    for sh in ({}, SHAPE):
        want = api.force_ij(xi, x, m, EPS, **kw, **sh)[0]
        p, a = over(xi)
        api.force_ij(p, x, m, EPS, out=(a, None), **kw, **sh)
        same(a, want, precision)
        want = api.force_jerk(x, v, m, EPS, **kw, **sh)[:2]
        (p, a), (w, j) = over(x), over(v)
        api.force_jerk(p, w, m, EPS, out=(a, j, None), **kw, **sh)
        same(a, want[0], precision)
        same(j, want[1], precision)
        want = api.force_jerk_ij(xi, vi, x, v, m, EPS, **kw, **sh)[:2]
        (p, a), (w, j) = over(xi), over(vi)
        api.force_jerk_ij(p, w, x, v, m, EPS, out=(a, j, None), **kw, **sh)
        same(a, want[0], precision)
        same(j, want[1], precision)
