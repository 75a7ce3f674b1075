"""Species steps where the wavefront forms can go wrong: hosts of one member to
several rows and chunks in one list (extents per run of lanes), dark-matter
counts around the tree's leaf and node sizes, baryon counts around a packet,
packets of several hosts, coincident dark matter (ties to the smaller index),
and a cell of several components next to one of a single one.  Labels are
exact."""
import numpy as np
import pytest

from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu

BITS = 16


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


def _hosts(dm, bar, scale, seed):
    """Hosts of dm[k] dark-matter and bar[k] baryon members, clumped, a few of
    them across the box faces, on coarse coordinates (coincident members)."""
    rng = np.random.default_rng(seed)
    size = np.array(dm) + np.array(bar)
    off = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    n = int(off[-1])
    gid = np.repeat(np.arange(len(size)), size)
    isb = np.concatenate([np.r_[np.zeros(d), np.ones(b)] for d, b in zip(dm, bar)]).astype(np.uint8)
    c = rng.integers(0, 1 << BITS, (3, len(size)))
    q = (c[:, gid] + 4 * np.rint(rng.normal(0, scale, (3, n))).astype(np.int64)) % (1 << BITS)
    v = np.rint(rng.normal(0, 3, (3, n))).astype(np.float32)
    perm = rng.permutation(n)
    qp, vp, ip = np.empty_like(q), np.empty_like(v), np.empty_like(isb)
    qp[:, perm], vp[:, perm], ip[perm] = q, v, isb
    mem = perm.astype(np.int32)
    for k in range(len(size)):
        mem[off[k]:off[k + 1]].sort()
    return qp.astype(np.uint32), vp, ip, off, mem


@pytest.mark.parametrize("dm,bar", [
    ([1, 1, 2, 3, 5] * 40, [0, 1, 1, 2, 3] * 40),
    ([63, 64, 65, 127, 128, 129, 1], [1, 15, 16, 17, 31, 33, 70]),
    ([4096, 4097, 5000, 64], [200, 64, 1, 300]),
    ([700, 30, 1100], [1500, 4000, 3]),
])
def test_assign_and_link(ctx, vr, ref, dm, bar):
    q, v, isb, off, mem = _hosts(dm, bar, 12.0, sum(dm))
    n = q.shape[1]
    rng = np.random.default_rng(n)
    sub = rng.integers(-1, 5, n).astype(np.int32)
    P, Pr = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(v), None, 1.0, 1.0, BITS), ref.Particles(q, v, None, 1.0, 1.0, BITS)
    ell = 10.0 / (1 << BITS)
    exp = ref.assign_baryons(Pr, off, mem, isb, sub, ell, 4.0)
    got = ctx.assign_baryons(P, dev_tensor(off), dev_tensor(mem), dev_tensor(isb), dev_tensor(sub), ell, 4.0)
    got = (got[0] if isinstance(got, tuple) else got).cpu().numpy()
    assert (got[mem] == exp[mem]).all()
    exp = ref.fof3d_dm(Pr, ell, isb)
    assert (ctx.fof3d_dm(P, ell, dev_tensor(isb)).cpu().numpy() == exp).all()


@pytest.mark.parametrize("more", [31, 32])
def test_assign_many(ctx, vr, ref, more):
    """Up to 786,431 baryons take four lanes each, more of them two."""
    q, v, isb, off, mem = _hosts([200] * 199 + [5], [3932] * 199 + [3932 + more], 12.0, more)
    n = q.shape[1]
    assert isb.sum() == 786400 + more
    sub = np.random.default_rng(n).integers(-1, 5, n).astype(np.int32)
    P, Pr = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(v), None, 1.0, 1.0, BITS), ref.Particles(q, v, None, 1.0, 1.0, BITS)
    ell = 10.0 / (1 << BITS)
    exp = ref.assign_baryons(Pr, off, mem, isb, sub, ell, 4.0)
    got, _ = ctx.assign_baryons(P, dev_tensor(off), dev_tensor(mem), dev_tensor(isb), dev_tensor(sub), ell, 4.0)
    assert (got.cpu().numpy()[mem] == exp[mem]).all()
