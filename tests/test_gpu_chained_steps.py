"""Integrator steps whose launches also start the next step, against the same steps taken one
at a time with separate evaluations: bitwise, since every operation and every order of
additions is the same.  Sizes on both sides of each limit of the chained launches."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import api, ics  # noqa: E402

DEV = "cuda"
EPS, DT = 0.02, 1.0 / 256.0


def state(n, seed):
    pos, vel, mass = ics.plummer(n, seed=seed)
    t = [torch.from_numpy(np.ascontiguousarray(v.T)).to(DEV) for v in (pos, vel)]
    return t[0], t[1], torch.from_numpy(mass.astype(np.float32)).to(DEV)


SIZES = [1, 255, 257, 2048, 4099, 8191, 8192, 8193, 10007, 65536, 65537]


@pytest.mark.parametrize("precision", ["comp", "plain"])
@pytest.mark.parametrize("n", SIZES)
def test_leapfrog_chain_equals_single_steps(n, precision):
    x0, v0, m = state(n, 11)
    xa, va = x0.clone(), v0.clone()
    acc, pot, traj = api.leapfrog(xa, va, m, EPS, DT, 3, with_pot=True, keep_trajectory=True,
                                  precision=precision)
    xb, vb = x0.clone(), v0.clone()
    a = api.force_f64(xb, m, EPS, precision=precision, with_pot=False)[0]
    assert torch.equal(traj[0], x0)
    for t in range(3):
        # One step per call starts with its own kick and drift and evaluates from scratch.
        a, p, _ = api.leapfrog(xb, vb, m, EPS, DT, 1, acc=a, init=False, with_pot=True,
                               precision=precision)
        assert torch.equal(traj[t + 1], xb)
    for u, w in ((xa, xb), (va, vb), (acc, a), (pot, p)):
        assert torch.equal(u, w)
    # The centre of the last evaluation is that of a separate call.
    f, q = api.force_f64(xa, m, EPS, precision=precision)
    assert torch.equal(acc, f) and torch.equal(pot, q)


@pytest.mark.parametrize("precision", ["comp", "plain"])
@pytest.mark.parametrize("n", [1, 200, 255, 2048, 2049, 4099, 8193, 65537])
def test_hermite_chain_equals_single_steps(n, precision):
    x0, v0, m = state(n, 12)
    a, j, _ = api.force_jerk(x0, v0, m, EPS, with_pot=False, precision=precision)
    sa = [x0.clone(), v0.clone(), a.clone(), j.clone()]
    api.hermite(sa[0], sa[1], m, EPS, DT, 3, acc=sa[2], jerk=sa[3], init=False,
                precision=precision)
    sb = [x0.clone(), v0.clone(), a.clone(), j.clone()]
    for _ in range(3):
        api.hermite(sb[0], sb[1], m, EPS, DT, 1, acc=sb[2], jerk=sb[3], init=False,
                    precision=precision)
    for u, w in zip(sa, sb):
        assert torch.equal(u, w)


@pytest.mark.parametrize("n", [300, 2049, 8193, 65537])
def test_chains_replayed_from_graphs(n):
    # Replays after eager work in between give the eager steps' state, every time.
    x0, v0, m = state(n, 13)
    acc = api.force_f64(x0, m, EPS, with_pot=False)[0]
    xe, ve, ae = x0.clone(), v0.clone(), acc.clone()
    g = api.LeapfrogGraph(x0, v0, m, EPS, DT, 2, acc)
    for _ in range(3):
        g.launch()
        api.force_f64(xe, m, EPS)
        ae = api.leapfrog(xe, ve, m, EPS, DT, 2, acc=ae, init=False)[0]
        torch.cuda.synchronize()
        assert torch.equal(x0, xe) and torch.equal(v0, ve) and torch.equal(acc, ae)


@pytest.mark.parametrize("sizes", [[256, 1, 0, 300, 4096], [256, 1, 0, 300, 4097]])
def test_batched_step_of_small_systems(sizes):
    # Up to 4096 particles per system, one launch does kick, drift, centre and conversion.
    off = np.concatenate([[0], np.cumsum(sizes)])
    parts = [state(n, 20 + k) for k, n in enumerate(sizes) if n]
    x, v = (torch.cat([p[c] for p in parts], dim=1).contiguous() for c in (0, 1))
    m = torch.cat([p[2] for p in parts])
    eps = torch.full((len(sizes),), EPS, dtype=torch.float32, device=DEV)
    plan = api.BatchPlan(off)
    acc, pot = plan.leapfrog(x, v, m, eps, DT, 2, with_pot=True)
    for k, n in enumerate(sizes):
        if not n:
            continue
        s = slice(int(off[k]), int(off[k + 1]))
        one = api.BatchPlan([0, n])
        xs, vs, ms = state(n, 20 + k)
        a1, p1 = one.leapfrog(xs, vs, ms, eps[:1], DT, 2, with_pot=True)
        for u, w in ((x[:, s], xs), (v[:, s], vs), (acc[:, s], a1), (pot[s], p1)):
            scale = max(float(w.abs().max()), 1e-300)
            assert float((u - w).abs().max()) <= 1e-11 * scale
