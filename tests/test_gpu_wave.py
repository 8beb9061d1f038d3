"""The wave engine at the edges of its shapes: i-groups of 64, 128 and 256 particles, stages
of 64 j-records, FP32 blocks of 64 and 128, one segment (outputs stored by the pair launch)
and several (finalize), for every accumulation mode, against the FP64 oracle with the
per-particle rounding bounds of the pair arithmetic."""
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
    pos, _, mass = ics.plummer(n, seed=seed, velocities=False)
    x = np.ascontiguousarray(pos.T.astype(np.float32))
    m = (mass * (1.0 + 0.5 * np.sin(np.arange(n)))).astype(np.float32)
    return x, m


def magnitudes(x, m, eps):
    return oracle.force_abs(x, m, x, eps, self_index=np.arange(len(m)))


def check(acc, pot, ref, ab, precision, n):
    check_acc(acc.cpu().numpy().T, ref[0], ab[0], precision, n)
    if pot is not None:
        check_pot(pot.cpu().numpy(), ref[1], ab[1], precision, n)


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("n", [1, 63, 65, 127, 129, 255, 257, 2049])
@pytest.mark.parametrize("ipl,jtile,nseg", [(1, 64, 1), (2, 128, 3), (4, 256, 2), (8, 64, 64)])
def test_force_shapes(precision, n, ipl, jtile, nseg):
    x, m = sphere(n, 70 + n)
    p, mm = torch.from_numpy(x).to(DEV), torch.from_numpy(m).to(DEV)
    x64, m64 = x.T.astype(np.float64), m.astype(np.float64)
    ref = oracle.force_all(x64, m64, float(np.float32(EPS)))
    ab = magnitudes(x64, m64, float(np.float32(EPS)))
    for with_pot in (True, False):
        acc, pot = api.force(p, mm, EPS, precision=precision, with_pot=with_pot, ipl=ipl,
                             jtile=jtile, nseg=nseg, jlanes=1)
        check(acc, pot, ref, ab, precision, n)


@pytest.mark.parametrize("n", [8192, 10007, 33000])
def test_segments_do_not_change_the_sums(n):
    # The FP32 blocks are the same for every split, so the results differ by the rounding of
    # FP64 (or FP32-pair) sums of them: at most a few 2^-47 of the sum of magnitudes.
    x, m = sphere(n, 5)
    p, mm = torch.from_numpy(x).to(DEV), torch.from_numpy(m).to(DEV)
    a0, p0 = api.force(p, mm, EPS)
    for ipl, nseg in ((1, 1), (2, 7), (4, 40)):
        a1, p1 = api.force(p, mm, EPS, ipl=ipl, jtile=128, nseg=nseg)
        scale = a0.abs().max()
        assert float((a1 - a0).abs().max() / scale) < 1e-11
        assert float(((p1 - p0) / p0).abs().max()) < 1e-11


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("ni,nj", [(1, 1), (1, 4000), (63, 65), (130, 2048), (300, 4097)])
def test_separate_sets_one_launch(precision, ni, nj):
    # Few i's: the waves of one block cover every j, also with no softening.
    rng = np.random.default_rng(ni * 7919 + nj)
    xi = rng.standard_normal((3, ni)).astype(np.float32)
    xj = rng.standard_normal((3, nj)).astype(np.float32)
    mj = rng.uniform(0.5, 1.5, nj).astype(np.float32)
    t = [torch.from_numpy(v).to(DEV) for v in (xi, xj, mj)]
    for eps in (0.0, EPS):
        acc, pot = api.force_ij(t[0], t[1], t[2], eps=eps, precision=precision)
        x64 = [v.T.astype(np.float64) for v in (xi, xj)]
        e = float(np.float32(eps))
        ra, rp = oracle.force_ij(x64[1], mj.astype(np.float64), x64[0], e)
        aa, ap = oracle.force_abs(x64[1], mj.astype(np.float64), x64[0], e)
        check_acc(acc.cpu().numpy().T, ra, aa, precision, nj)
        check_pot(pot.cpu().numpy(), rp, ap, precision, nj)


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("sizes", [[256, 300, 64, 1, 1500], [9000, 200, 5000], [17000, 31]])
def test_batched_open_shape(precision, sizes):
    # The open shape's items: whole systems (outputs stored by the pair launch) and systems in
    # several segments, one plan holding both.
    off = np.concatenate([[0], np.cumsum(sizes)])
    xs = [sphere(n, 90 + n) for n in sizes]
    x = np.concatenate([a for a, _ in xs], axis=1)
    m = np.concatenate([b for _, b in xs])
    eps = np.full(len(sizes), EPS, dtype=np.float32)
    plan = api.BatchPlan(off, precision=precision)
    acc, pot = plan.force(*[torch.from_numpy(v).to(DEV) for v in (x, m, eps)])
    for k, n in enumerate(sizes):
        s = slice(int(off[k]), int(off[k + 1]))
        x64, m64 = x[:, s].T.astype(np.float64), m[s].astype(np.float64)
        ref = oracle.force_all(x64, m64, float(eps[k]))
        ab = magnitudes(x64, m64, float(eps[k]))
        check(acc[:, s], pot[s], ref, ab, precision, n)


@pytest.mark.parametrize("n", [1, 64, 129, 1000, 2048, 2049, 5000, 17000])
def test_jerk_and_adjoint_splits_agree(n):
    # One launch (few j's) or segments and a finalize, 1 or 2 i's per lane: the FP32 blocks are
    # the same, so the results differ by the rounding of FP64 sums of them, at most a few
    # 2^-47 of the sum of magnitudes.
    x, m = sphere(n, 6)
    rng = np.random.default_rng(n)
    p, mm = torch.from_numpy(x).to(DEV), torch.from_numpy(m).to(DEV)
    v = torch.from_numpy(rng.standard_normal((3, n)).astype(np.float32)).to(DEV)
    ref = api.force_jerk(p, v, mm, EPS)
    k = max(1, n // 3)
    pi, vi = p[:, :k].contiguous(), v[:, :k].contiguous()
    ref_ij = api.force_jerk_ij(pi, vi, p, v, mm, EPS)
    p64 = p.double()
    g = torch.from_numpy(rng.standard_normal((3, n))).to(DEV)
    gp = torch.from_numpy(rng.standard_normal(n)).to(DEV)

    def vjp(**kw):
        gx, gm = torch.empty_like(g), torch.empty_like(gp)
        _lib.nbody_force_vjp_f64(n, p64.data_ptr(), mm.data_ptr(), EPS, g.data_ptr(), gp.data_ptr(),
                                 gx.data_ptr(), gm.data_ptr(), api.make_opts(**kw), api.stream_ptr())
        return gx, gm

    ref_vjp = vjp()
    for ipl, nseg in ((1, 1), (2, 3), (4, 16)):
        kw = {"ipl": ipl, "jtile": 128, "nseg": nseg}
        for a, b in zip(ref + ref_ij + ref_vjp,
                        api.force_jerk(p, v, mm, EPS, **kw)
                        + api.force_jerk_ij(pi, vi, p, v, mm, EPS, **kw) + vjp(**kw)):
            assert float((a - b).abs().max()) <= 1e-11 * max(float(a.abs().max()), 1e-300)


@pytest.mark.parametrize("precision", ["comp", "plain"])
@pytest.mark.parametrize("n", [3000, 4099, 9000])
def test_waves_that_end_together(precision, n):
    # One to five waves per SIMD: only priorities differ from a launch of more waves (segments
    # asked for), so the sums differ by the rounding of FP64 (PLAIN: of 2 against ceil(n / 256)
    # FP32 segments, at most n 2^-24 of the sum of magnitudes).
    x, m = sphere(n, 6)
    v = np.ascontiguousarray(x[::-1])
    p, w, mm = (torch.from_numpy(t).to(DEV) for t in (x, v, m))
    one = api.force_jerk(p, w, mm, EPS, precision=precision)
    two = api.force_jerk(p, w, mm, EPS, precision=precision, ipl=2, jtile=128,
                         nseg=2 if precision == "plain" else 64)
    tol = 1e-11 if precision == "comp" else n * 2.0 ** -24
    for a, b in zip(one, two):
        assert float((a - b).abs().max() / a.abs().max()) < tol
