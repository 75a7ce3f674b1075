"""Features of the surrogate where its tables can go wrong: the smallest grid
(16 fine and 4 coarse cells a side, whose windows wrap), members alone in their
cells, thousands in one cell (sums of more and of fewer than eight members), and
tables as full as they get.  BF16 features differ by one unit in the last place
at most, where the oracle's value lies on a rounding boundary."""
import numpy as np
import pytest

from oracle import surrogate as S
from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


@pytest.mark.parametrize("bits,cell_bits", [(8, 4), (12, 4), (21, 12)])
@pytest.mark.parametrize("m,spread", [(1, 0.3), (7, 0.01), (768, 0.5), (3000, 0.0), (6000, 0.02), (20000, 0.25)])
def test_features(ctx, vr, bits, cell_bits, m, spread):
    rng = np.random.default_rng(m + bits)
    size = 1 << bits
    q = np.rint(size * (0.01 + spread * rng.normal(size=(3, m)))).astype(np.int64) % size
    q = q.astype(np.uint32)
    v = rng.normal(0, 100, (3, m)).astype(np.float32)
    vbar = rng.normal(0, 20, (3, m)).astype(np.float32)
    a = rng.normal(size=(m, 3, 3))
    cov = 1e4 * (np.eye(3) + 0.2 * np.einsum("nij,nkj->nik", a, a))
    sigma = np.stack([cov[:, 0, 0], cov[:, 1, 1], cov[:, 2, 2], cov[:, 0, 1], cov[:, 0, 2], cov[:, 1, 2]]).astype(np.float32)
    rho = (1e10 * np.exp(rng.normal(size=m))).astype(np.float32)
    mem = np.sort(rng.permutation(m)).astype(np.int32)
    exp = S.bf16_bits(S.features(q, v, mem, vbar, sigma, rho, 32, cell_bits, 100.0, bits))
    P = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(v), None, 1.0, 100.0, bits)
    got = ctx.rs_features(P, dev_tensor(np.array([0, m], np.int32)), dev_tensor(mem), dev_tensor(vbar), dev_tensor(sigma),
                          dev_tensor(rho), 32, cell_bits).cpu().numpy().view(np.uint16)
    assert got.shape == exp.shape
    ge, ee = S.bf16_from_bits(got), S.bf16_from_bits(exp)
    assert (np.isnan(ge) == np.isnan(ee)).all()
    ok = ~np.isnan(ee) & ~((ge == 0) & (ee == 0))
    # values next to zero: the terms' rounding, not the value's, is what differs
    near = np.abs(ge - ee) <= 1e-9
    diff = np.abs(got.astype(np.int32) - exp.astype(np.int32))
    assert ((diff <= 1) | near)[ok].all()
    assert (diff[ok & ~near] != 0).mean() <= 5e-3 if (ok & ~near).any() else True
