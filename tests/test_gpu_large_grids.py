"""Calls whose work needs more threads than one launch can have (2^32 - 1 along a dimension):
a batch of more than 2^24 systems, and more than 2^28 i-particles against a j-set that a block
of 16 waves shares."""
import ctypes

import numpy as np
import pytest

import oracle
from bounds import check_acc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import _lib, api  # noqa: E402

DEV = "cuda"


def test_batch_of_many_pairs():
    # Two-particle systems: a_0 = m_1 d / s^3 and a_1 = -m_0 d / s^3 in closed form.
    nsys = (1 << 24) + 5
    off = np.arange(nsys + 1, dtype=np.int64) * 2
    h = ctypes.c_void_p()
    opts = api.make_opts()
    st = _lib.load().nbody_plan_create_batched(
        nsys, off.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), ctypes.byref(opts),
        ctypes.byref(h))
    assert st == _lib.NBODY_OK, _lib.nbody_last_error()
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(5)
        n = 2 * nsys
        x = torch.randn((3, n), generator=g, device=DEV)
        m = torch.rand(n, generator=g, device=DEV) + 0.5
        eps = torch.full((nsys,), 0.25, device=DEV)
        acc = torch.full((3, n), float("nan"), dtype=torch.float64, device=DEV)
        _lib.nbody_force_batched(h.value, x.data_ptr(), m.data_ptr(), eps.data_ptr(),
                                 acc.data_ptr(), None, api.stream_ptr())
        d = (x[:, 1::2] - x[:, 0::2]).double()
        r3 = ((d * d).sum(0) + 0.0625) ** -1.5
        # One pair term: 18 roundings of 2^-24 at most (bounds.py).
        tol = 18 * 2.0 ** -24
        for k, sign in ((0, 1.0), (1, -1.0)):
            want = sign * m[1 - k::2].double() * r3 * d
            assert bool(((acc[:, k::2] - want).abs() <= tol * want.abs() + 1e-300).all())
    finally:
        torch.cuda.synchronize()
        _lib.nbody_plan_destroy(h.value)


def test_many_i_particles():
    ni, nj, eps = 1 << 28, 8192, 0.5
    g = torch.Generator(device=DEV)
    g.manual_seed(6)
    xi = torch.rand((3, ni), generator=g, device=DEV)
    xj = torch.rand((3, nj), generator=g, device=DEV)
    mj = torch.rand(nj, generator=g, device=DEV) / nj
    acc, _ = api.force_ij(xi, xj, mj, eps=eps, with_pot=False, ipl=1, jtile=128)
    pick = torch.tensor([0, 63, 64, ni // 3, ni // 2 - 1, ni // 2, ni - 65, ni - 64, ni - 1],
                        device=DEV)
    f = lambda t: np.ascontiguousarray(t.cpu().numpy().astype(np.float64).T)
    x64, j64, m64 = f(xi[:, pick]), f(xj), mj.cpu().numpy().astype(np.float64)
    ref, _ = oracle.force_ij(j64, m64, x64, eps)
    ab, _ = oracle.force_abs(j64, m64, x64, eps)
    check_acc(f(acc[:, pick]), ref, ab, "comp", nj)
    assert bool(torch.isfinite(acc).all())
