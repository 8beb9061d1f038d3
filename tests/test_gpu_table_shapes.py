"""A grid-engine entry of the tuning table runs the launch that the same values in a call's
options run: bitwise the same results, for every kernel that the table serves."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_astro_ph_0703100_amd import _lib, api, ics  # noqa: E402

DEV = "cuda"
EPS = 0.02


@pytest.fixture(autouse=True)
def committed_table():
    yield
    _lib.nbody_tune_reset()
    _lib.nbody_tune_load(_lib.TUNING_PATH)


@pytest.mark.parametrize("precision", ["comp", "fp64red", "plain"])
@pytest.mark.parametrize("shape", [(1, 64, 8), (2, 128, 3), (1, 128, 0), (0, 64, 5), (4, 256, 0),
                                   (8, 512, 6), (0, 128, 0)])
@pytest.mark.parametrize("n", [3001, 20011])
def test_entry_and_options_run_the_same_launch(precision, shape, n):
    pos, vel, mass = ics.plummer(n, seed=4)
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).to(DEV)
    x, v, m = f(pos.T), f(vel.T), f(mass)
    x64 = x.double()
    g = torch.randn((3, n), dtype=torch.float64, device=DEV)
    off = [0, 5, 1000, n]
    eps = torch.full((3,), EPS, device=DEV)

    def vjp(**kw):
        gx, gm = torch.empty_like(g), torch.empty(n, dtype=torch.float64, device=DEV)
        _lib.nbody_force_vjp(n, x.data_ptr(), m.data_ptr(), EPS, g.data_ptr(), None,
                             gx.data_ptr(), gm.data_ptr(),
                             api.make_opts(precision=precision, **kw), api.stream_ptr())
        return gx, gm

    def batch(**kw):
        plan = api.BatchPlan(off, precision=precision, **kw)
        out = plan.force(x, m, eps)
        plan.close()
        return out

    def results(sh, bsh):
        return [*api.force(x, m, EPS, precision=precision, **sh),
                *api.force_f64(x64, m, EPS, precision=precision, centre="tile", **sh),
                *api.force_jerk(x, v, m, EPS, precision=precision, **sh), *vjp(**sh),
                *batch(**bsh)]

    ipl, jtile, nseg = shape
    _lib.nbody_tune_reset()
    asked = results({"ipl": ipl, "jtile": jtile, "nseg": nseg, "jlanes": 1},
                    {"ipl": ipl, "jtile": jtile})
    for k in _lib.KERNELS.values():
        for size in (n, n // 3):  # batches go by their mean size
            _lib.nbody_tune_set(k, _lib.PRECISIONS[precision], size, ipl, jtile, nseg)
    assert _lib.nbody_tune_get(_lib.NBODY_KERNEL_JERK, _lib.PRECISIONS[precision], n) == \
        (ipl, jtile, nseg, 1, 0)
    for a, b in zip(asked, results({}, {})):
        assert torch.equal(a, b)
