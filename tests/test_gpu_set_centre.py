"""The whole-set force from FP64 positions with the centre that its own launch sums: potentials
and accelerations of asked lanes and tiles within the rounding bounds of the pair arithmetic,
against the oracle on the same FP32 positions.  The coordinates are multiples of 2^-20 below
2^8, so their FP64 sum is exact in any order and fp32(x - c) is the library's own input."""
import numpy as np
import pytest

import oracle
from bounds import C_POT, U, adds, check_acc, check_pot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import api, ics  # noqa: E402

DEV = "cuda"
EPS = 0.02


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("jlanes,jtile", [(32, 256), (32, 1024), (64, 256), (64, 1024)])
@pytest.mark.parametrize("n", [3, 258, 2300, 4097, 8192])
def test_potentials_and_accelerations(precision, jlanes, jtile, n):
    pos, _, mass = ics.plummer(n, seed=4)
    pos = np.round((pos + np.array([100.0, -30.0, 7.0])) * 2.0 ** 20) / 2.0 ** 20
    m = (mass * (1.0 + 0.5 * np.sin(np.arange(n)))).astype(np.float32)
    x = (pos - pos.sum(axis=0) / n).astype(np.float32).astype(np.float64)
    m64, eps = m.astype(np.float64), float(np.float32(EPS))
    ref = oracle.force_all(x, m64, eps)
    ab = oracle.force_abs(x, m64, x, eps, self_index=np.arange(n))
    p64 = torch.from_numpy(np.ascontiguousarray(pos.T)).to(DEV)
    mm = torch.from_numpy(m).to(DEV)
    kw = dict(precision=precision, jlanes=jlanes, jtile=jtile, ipl=1)
    for pot in (True, False):
        acc, phi = api.force_f64(p64, mm, EPS, with_pot=pot, **kw)
        check_acc(acc.cpu().numpy().T, ref[0], ab[0], precision, n)
        if pot:
            check_pot(phi.cpu().numpy(), ref[1], ab[1], precision, n)
    # A particle's own record in its potential is far outside the bound.
    bound = (C_POT + adds(precision, n)) * U * ab[1]
    assert (m64 / eps > 4.0 * bound).all()
