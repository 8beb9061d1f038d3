"""Shapes that a caller asks for, at the edges of the rules that launch them: records per lane
for launches of few waves, j-segments of few FP32 blocks, one launch or several segments, PLAIN
blocks of one and four waves, and the engine of 32 lanes per particle.  Against the FP64 oracle
with the per-particle rounding bounds of the pair arithmetic."""
import numpy as np
import pytest

import oracle
from bounds import check_acc, check_pot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import api, ics  # noqa: E402

DEV = "cuda"
EPS = 0.02
MODES = ["comp", "fp64red", "plain"]


def sphere(n, seed):
    pos, _, mass = ics.plummer(n, seed=seed, velocities=False)
    m = (mass * (1.0 + 0.5 * np.sin(np.arange(n)))).astype(np.float32)
    return np.ascontiguousarray(pos.T), m


def reference(x, m):
    x64, m64 = x.T.astype(np.float64), m.astype(np.float64)
    eps = float(np.float32(EPS))
    return (oracle.force_all(x64, m64, eps),
            oracle.force_abs(x64, m64, x64, eps, self_index=np.arange(len(m))))


def check(got, want, precision, n):
    (acc, pot), (ref, ab) = got, want
    check_acc(acc.cpu().numpy().T, ref[0], ab[0], precision, n)
    if pot is not None:
        check_pot(pot.cpu().numpy(), ref[1], ab[1], precision, n)


@pytest.mark.parametrize("precision", MODES)
@pytest.mark.parametrize("n", [65, 1024, 1025, 2048, 2049, 5000])
def test_records_and_segments(precision, n):
    x, m = sphere(n, 11)
    x = x.astype(np.float32)
    p, mm = torch.from_numpy(x).to(DEV), torch.from_numpy(m).to(DEV)
    want = reference(x, m)
    for ipl, jtile, nseg in ((0, 64, 0), (2, 64, 0), (4, 128, 0), (8, 512, 0), (1, 64, 3),
                             (1, 64, 17), (1, 64, 1000), (2, 128, 9), (4, 256, 5)):
        for pot in (True, False):
            check(api.force(p, mm, EPS, precision=precision, with_pot=pot, ipl=ipl, jtile=jtile,
                            nseg=nseg, jlanes=1), want, precision, n)


@pytest.mark.parametrize("precision", MODES)
@pytest.mark.parametrize("ni,nj,nseg", [(64, 1024, 0), (64, 1025, 0), (16320, 2048, 0),
                                        (16384, 2048, 0), (200, 4096, 3), (200, 4096, 4),
                                        (200, 4096, 7), (2048, 8192, 32), (2049, 8192, 32)])
def test_separate_sets(precision, ni, nj, nseg):
    rng = np.random.default_rng(ni + nj)
    xi = rng.standard_normal((3, ni)).astype(np.float32)
    xj = rng.standard_normal((3, nj)).astype(np.float32)
    mj = rng.uniform(0.5, 1.5, nj).astype(np.float32)
    t = [torch.from_numpy(v).to(DEV) for v in (xi, xj, mj)]
    kw = {"nseg": nseg, "jtile": 128} if nseg else {}
    acc, pot = api.force_ij(*t, eps=EPS, precision=precision, **kw)
    pick = np.unique(np.linspace(0, ni - 1, 200).astype(np.int64))
    xs, x64, m64 = (v.T.astype(np.float64) for v in (xi[:, pick], xj, mj))
    eps = float(np.float32(EPS))
    ref, ab = oracle.force_ij(x64, m64, xs, eps), oracle.force_abs(x64, m64, xs, eps)
    check_acc(acc.cpu().numpy().T[pick], ref[0], ab[0], precision, nj)
    check_pot(pot.cpu().numpy()[pick], ref[1], ab[1], precision, nj)


@pytest.mark.parametrize("precision", MODES)
@pytest.mark.parametrize("jtile", [256, 1024, 2048])
@pytest.mark.parametrize("n", [511, 512, 2047, 2048, 2049, 4095, 4096, 4097])
def test_lanes_of_small_systems(precision, jtile, n):
    # FP32 positions (either engine of 32 lanes), and FP64 positions in their own place (a
    # conversion and the FP32 launch) and apart (one launch): the same sums.
    x, m = sphere(n, 12)
    mm = torch.from_numpy(m).to(DEV)
    kw = dict(precision=precision, ipl=1, jtile=jtile, jlanes=32)
    x32 = x.astype(np.float32)
    check(api.force(torch.from_numpy(x32).to(DEV), mm, EPS, **kw), reference(x32, m), precision, n)
    x64 = torch.from_numpy(x).to(DEV)
    acc, pot = api.force_f64(x64, mm, EPS, **kw)
    buf, p = x64.clone(), torch.empty_like(pot)
    api.force_f64(buf, mm, EPS, out=(buf, p), **kw)
    assert torch.equal(buf, acc) and torch.equal(p, pot)


@pytest.mark.parametrize("sizes,ipl,want,per_iteration", [
    ([300, 1000], 0, 1, 16), ([300, 1000], 8, 1, 16), ([20000, 33, 7], 2, 2, 8),
    ([40000, 64], 8, 4, 8)])
def test_plan_info_describes_the_launch(sizes, ipl, want, per_iteration):
    # Records per lane of the launch (an asked number is an upper limit), one block per item,
    # and pairs with the i-groups filled and the j's in whole iterations.
    off = np.concatenate([[0], np.cumsum(sizes)])
    plan = api.BatchPlan(off, ipl=ipl, jtile=128)
    info = plan.info()
    plan.close()
    assert info["ipl"] == want and info["blocks"] == info["items"]
    group = 64 * want
    pairs = items = 0
    for n in sizes:
        segs = -(-n // 4096)
        per = -(-(-(-n // 128)) // segs) * 128
        lens = [min(per, n - s) for s in range(0, n, per)]
        items += -(-n // group) * len(lens)
        pairs += -(-n // group) * group * sum(-(-j // per_iteration) * per_iteration for j in lens)
    assert info["items"] == items and info["padded_pairs"] == pairs
