"""The persistent unbinding schedule at the sizes where its tiles, items and
selections can go wrong: groups around multiples of 64 members and of the
items' column ranges, particle masses, eps = 0 with coincident members, more
candidates for the minimum than are refined one by one, and more members at
one distance than the frame's list holds.  phi's tolerance is the bound of its
FP32 runs (64 additions, half an ulp each, 64 * 2^-24 = 4e-6, and terms rounded
to two ulp), and as much again for what incremental passes subtract."""
import numpy as np
import pytest

from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu

BITS, BOX = 21, 100.0
RTOL = 2 * (64 * 2.0 ** -24 + 2 * 2.0 ** -23)


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


def _case(sizes, masses, clump, seed):
    """Gaussian groups (some across the box faces) with a fifth of the members,
    none of them in the inner half, too fast to be bound; a fraction `clump` of
    each group on one point."""
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(off[-1])
    gid = np.repeat(np.arange(len(sizes)), sizes)
    centre = rng.integers(0, 1 << BITS, (3, len(sizes)))
    x = np.rint(rng.normal(0, 3000.0, (3, n))).astype(np.int64)
    x[:, rng.random(n) < clump] = 0
    q = ((centre[:, gid] + x) % (1 << BITS)).astype(np.uint32)
    v = rng.normal(0, 0.05, (3, n)).astype(np.float32)
    v[0, (rng.random(n) < 0.4) & ((x * x).sum(0) > 3 * 2400 ** 2)] += 1e4
    mass = rng.uniform(0.5, 1.5, n).astype(np.float32) if masses else None
    mem = rng.permutation(n).astype(np.int32)  # groups interleaved in the particle arrays
    for g in range(len(sizes)):
        mem[off[g]:off[g + 1]].sort()
    qp, vp = np.empty_like(q), np.empty_like(v)
    qp[:, mem], vp[:, mem] = q, v
    return qp, vp, mass, off, mem


@pytest.mark.parametrize("sizes,masses,eps,clump,jchunk", [
    ([20, 63, 64, 65, 127, 128, 129, 191, 193, 255, 257], False, 0.05, 0.0, 4096),
    ([20, 63, 64, 65, 127, 128, 129, 191, 193, 255, 257], True, 0.05, 0.0, 256),
    ([4095, 4096, 4097, 4160, 2049], False, 0.05, 0.0, 4096),
    ([1023, 1024, 1025, 1088], True, 0.02, 0.0, 256),
    ([64, 65, 640, 1000], False, 0.0, 0.3, 256),
    ([64, 65, 640, 1000], True, 0.0, 0.3, 256),
    ([4097, 3000, 130, 60], False, 0.05, 0.6, 4096),
])
def test_tiles_and_selection(ctx, vr, ref, sizes, masses, eps, clump, jchunk):
    q, vel, mass, off, mem = _case(sizes, masses, clump, seed=sum(sizes))
    P = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(vel), None if mass is None else dev_tensor(mass), 1.0, BOX,
                     BITS)
    Pr = ref.Particles(q, vel, mass, 1.0, BOX, BITS)
    exp = ref.unbind(Pr, off, mem, 1.0, eps)
    saved = ctx.get_tune("unbind_jchunk")
    try:
        ctx.tune("unbind_jchunk", jchunk)
        got = ctx.unbind(P, dev_tensor(off), dev_tensor(mem), 1.0, eps, persistent=1)
    finally:
        ctx.tune("unbind_jchunk", saved)
    clean = exp["min_margin"] > 1e-5
    assert clean.all()
    assert (got["bound"].cpu().numpy() == exp["bound"]).all()
    assert (got["iters"].cpu().numpy() == exp["iters"]).all()
    phi = got["phi"].cpu().numpy()
    fin = np.isfinite(exp["phi"])
    assert (np.isfinite(phi) == fin).all()
    np.testing.assert_allclose(phi[fin], exp["phi"][fin], rtol=RTOL)
