"""The relaxed stage of the paper's linker and the fit of L where the wavefront
forms can go wrong: grids of two cells a side (the 27 neighbours repeat), four
and many; cells without participants around; more than 64 candidates a cell;
and fits with fewer bins than a wavefront, about 64 and many.  Labels and
rounds are exact."""
import numpy as np
import pytest

from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


@pytest.mark.parametrize("bits,ell,scale", [(8, 0.3, 30.0), (8, 0.13, 12.0), (12, 0.004, 12.0), (21, 2e-4, 500.0)])
@pytest.mark.parametrize("clumps", [1, 6])
def test_growth_and_joins(ctx, vr, ref, bits, ell, scale, clumps):
    rng = np.random.default_rng(bits + clumps)
    n, size = 3000, 1 << bits
    c = rng.integers(0, size, (3, clumps))
    q = (c[:, rng.integers(0, clumps, n)] + np.rint(rng.normal(0, scale, (3, n))).astype(np.int64)) % size
    q = q.astype(np.uint32)
    v = (rng.normal(0, 1.0, (3, n)) + 3.0).astype(np.float32)
    vbar = rng.normal(0, 0.1, (3, n)).astype(np.float32)
    L = rng.normal(2.5, 1.0, n).astype(np.float32)
    host = np.where(rng.random(n) < 0.02, -1, 0).astype(np.int32)
    P, Pr = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(v), None, 1.0, 1.0, bits), ref.Particles(q, v, None, 1.0, 1.0, bits)
    lab = ref.fof_sub(Pr, host, 1, vbar, 0.5 * ell, L, 3.0, 2.0, theta_op=0.5)
    exp = ref.sub_grow(Pr, host, 1, vbar, L, lab, 0.5 * ell, 3.0, gamma_L=1.5, gamma_x=2.0, Vr=2.0, theta_op=0.5, n_min=5)
    got = ctx.sub_grow(P, dev_tensor(host), 1, dev_tensor(vbar), dev_tensor(L), dev_tensor(lab), 0.5 * ell, 3.0,
                       gamma_L=1.5, gamma_x=2.0, Vr=2.0, theta_op=0.5, n_min=5)
    assert (got[0].cpu().numpy() == exp[0]).all()
    assert int(got[1]) == int(exp[1])


@pytest.mark.parametrize("n,width", [(300, 0.5), (4000, 0.05), (60000, 1.0 / 32), (60000, 1.0 / 64)])
def test_fit_bins(ctx, ref, n, width):
    """Bins from a handful to several a lane; the fit's tolerance is the one
    the fit is held to elsewhere (1e-6 of the golden section's bracket)."""
    rng = np.random.default_rng(n)
    R = (0.2 + np.where(rng.random(n) < 0.5, -0.9, 0.7) * np.abs(rng.normal(0, 1, n))).astype(np.float32)
    off, mem = np.array([0, n], np.int32), np.arange(n, dtype=np.int32)
    kw = dict(width=width, peak_min=8)
    exp = ref.ell_fit(R, off, mem, **kw)
    got = ctx.ell_fit(dev_tensor(R), dev_tensor(off), dev_tensor(mem), **kw)
    assert (got["status"].cpu().numpy() == exp["status"]).all() and (got["merge"].cpu().numpy() == exp["merge"]).all()
    np.testing.assert_allclose(got["fit"].cpu().numpy(), exp["fit"], rtol=1e-6, atol=1e-6)
