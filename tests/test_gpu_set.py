"""The force with every record in the LDS of one compute unit, at the edges of its shapes:
chunks of 256 records, 1 or 2 particles per wave, 4 to 16 waves, tiles (whole, in pairs, the
last one), 32 and 64 lanes per particle, the largest size; FP64 positions with the centre
summed by the same launch against the separate centre and conversion."""
import numpy as np
import pytest

import oracle
from bounds import check_acc, check_pot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import _lib, api, ics  # noqa: E402

DEV = "cuda"
EPS = 0.02


def sphere(n, seed):
    pos, vel, mass = ics.plummer(n, seed=seed)
    m = (mass * (1.0 + 0.5 * np.sin(np.arange(n)))).astype(np.float32)
    return np.ascontiguousarray(pos.T), np.ascontiguousarray(vel.T), m


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("n", [1, 2, 1025, 2048, 2049, 3073, 4095, 4096, 4097, 5121, 6144, 6145,
                               7168, 8191])
def test_force_sizes(precision, n):
    pos, _, m = sphere(n, 30 + n % 7)
    p, mm = torch.from_numpy(pos.astype(np.float32)).to(DEV), torch.from_numpy(m).to(DEV)
    x64 = np.ascontiguousarray(pos.astype(np.float32).T.astype(np.float64))
    m64 = m.astype(np.float64)
    eps = float(np.float32(EPS))
    ref = oracle.force_all(x64, m64, eps)
    ab = oracle.force_abs(x64, m64, x64, eps, self_index=np.arange(n))
    # FP64 positions that FP32 holds, without a centre: the same pairs.
    p64 = p.double()
    for pot in (True, False):
        for acc, phi in (api.force(p, mm, EPS, precision=precision, with_pot=pot),
                         api.force_f64(p64, mm, EPS, precision=precision, with_pot=pot,
                                       centre="none")):
            check_acc(acc.cpu().numpy().T, ref[0], ab[0], precision, n)
            if pot:
                check_pot(phi.cpu().numpy(), ref[1], ab[1], precision, n)


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("jlanes,jtile", [(32, 256), (32, 1024), (64, 256), (64, 1024)])
@pytest.mark.parametrize("n", [3, 258, 2300, 8192])
def test_asked_shapes(precision, jlanes, jtile, n):
    pos, _, m = sphere(n, 4)
    p64, mm = torch.from_numpy(pos).to(DEV), torch.from_numpy(m).to(DEV)
    kw = dict(precision=precision, jlanes=jlanes, jtile=jtile, ipl=1)
    a, p = api.force_f64(p64, mm, EPS, **kw)
    # In place, the centre and the conversion are a launch of their own.
    buf = p64.clone()
    api.force_f64(buf, mm, EPS, out=(buf, None), **kw)
    assert torch.equal(buf, a)
    c = p64.cpu().numpy().mean(axis=1, keepdims=True)
    x = np.ascontiguousarray((pos - c).T)
    eps = float(np.float32(EPS))
    ref = oracle.force_all(x, m.astype(np.float64), eps)
    scale = np.abs(ref[0]).max()
    # FP32 positions and pairs: errors of a few 2^-24 of the field, times the softened
    # gradient (|x| / EPS < 2^14 at most); far below a wrong or missing record.
    assert np.abs(a.cpu().numpy().T - ref[0]).max() < 1e-3 * scale


@pytest.mark.parametrize("n,steps", [(1, 2), (300, 3), (2048, 4), (2049, 5), (4500, 3), (8191, 2)])
@pytest.mark.parametrize("precision", ["comp", "plain"])
def test_steps_in_a_small_workspace(precision, n, steps):
    # A workspace of the stated size has no room for a second set of positions: the steps then
    # convert and evaluate in two launches, with the same result.
    pos, vel, m = sphere(n, 9)
    mm = torch.from_numpy(m).to(DEV)
    state = [torch.from_numpy(v).to(DEV) for v in (pos, vel)]
    opts = api.make_opts(precision=precision)
    size = _lib.nbody_workspace_size(n, opts)
    out = []
    for extra in (None, 0, 3 * 8 * n):
        x, v = state[0].clone(), state[1].clone()
        kw = {}
        if extra is not None:
            kw["workspace"] = torch.empty(size + extra, dtype=torch.uint8, device=DEV)
        acc, pot, traj = api.leapfrog(x, v, mm, EPS, 1.0 / 64, steps, with_pot=True,
                                      keep_trajectory=True, precision=precision, **kw)
        assert torch.equal(traj[-1], x)
        out.append((x, v, acc, pot, traj))
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert torch.equal(a, b)
