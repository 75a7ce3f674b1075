"""The neighbour tree and search at the sizes where they can go wrong: hosts
around multiples of a leaf and of a bucket, neighbour counts at the limits of
each kernel form, more coincident members than a query's lists hold, and
subsets whose wavefronts span hosts."""
import numpy as np
import pytest

from paper_1902_01010_amd import synth
from tests.gpu_common import R_agrees, both, dev_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


def _hosts(rng, sizes, box=1.0, extent=0.02, masses=False):
    """Gaussian blobs of the given sizes as one workload and its host table."""
    n = int(sum(sizes))
    pos = np.empty((3, n))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    for h, s in enumerate(sizes):
        c = rng.random((3, 1)) * box
        pos[:, off[h]:off[h + 1]] = c + rng.normal(0, extent, (3, s))
    vel = rng.normal(0, 100.0, (3, n))
    x = np.mod(pos, box).astype(np.float32)
    x[x >= np.float32(box)] = 0
    m = (0.5 + rng.random(n)).astype(np.float32) if masses else None
    w = synth.Workload("blobs", x, vel.astype(np.float32), m, 1.0, box, 21, {}, {})
    vbar = rng.normal(0, 10.0, (3, n)).astype(np.float32)
    s2 = rng.uniform(0.5e4, 2e4, (3, n))
    sigma = np.concatenate([s2, 0.1 * s2]).astype(np.float32)
    return w, off, np.arange(n, dtype=np.int32), vbar, sigma


def _check(ctx, vr, ref, case, n_se, n_v, subset=None):
    w, off, mem, vbar, sigma = case
    P, Pr = both(ctx, vr, ref, w)
    exp = ref.local_vdensity(Pr, off, mem, vbar, sigma, n_se, n_v, subset=subset)["R"]
    got = ctx.local_vdensity(P, dev_tensor(off), dev_tensor(mem), dev_tensor(vbar), dev_tensor(sigma), n_se, n_v,
                             subset=None if subset is None else dev_tensor(subset)).cpu().numpy()
    assert np.isfinite(exp).any()
    R_agrees(got, exp)


@pytest.mark.parametrize("n_se,n_v,masses", [(2, 2, False), (31, 8, True), (32, 32, False), (33, 8, False), (64, 64, True),
                                             (65, 3, False), (128, 32, True), (129, 32, False), (256, 32, True)])
def test_leaf_and_bucket_edges(ctx, vr, ref, n_se, n_v, masses):
    """Hosts of exactly n_se members, one leaf more or less, and around 2048
    (a full bucket) and 4096 (two)."""
    rng = np.random.default_rng(n_se)
    sizes = [n_se, n_se + 1] + [s for s in (63, 64, 65, 257, 2047, 2048, 2049, 4097) if s >= n_se]
    saved = ctx.get_tune("knn_leaf")
    try:
        for leaf in (16, 256):  # buckets of 256 and 2048 members
            ctx.tune("knn_leaf", leaf)
            _check(ctx, vr, ref, _hosts(rng, sizes, masses=masses), n_se, n_v)
    finally:
        ctx.tune("knn_leaf", saved)


@pytest.mark.parametrize("n_se,n_v", [(32, 8), (48, 16), (256, 32)])
def test_coincident_members_overflow_the_lists(ctx, vr, ref, n_se, n_v):
    """700 members at one point: every query there has more members at its
    radius than its lists hold; ties break by particle index."""
    rng = np.random.default_rng(6)
    case = _hosts(rng, [1500, 900], masses=True)
    case[0].x[:, 200:900] = case[0].x[:, 200:201]
    case[0].x[:, 1500:1540] = case[0].x[:, 1500:1501]
    _check(ctx, vr, ref, case, n_se, n_v)


def test_equal_velocities(ctx, vr, ref):
    """Velocity ties at the n_v-th neighbour, and n_v members at distance zero."""
    rng = np.random.default_rng(7)
    case = _hosts(rng, [2000])
    case[0].v[:, ::3] = np.round(case[0].v[:, ::3] / 80) * 80
    case[0].v[:, :60] = case[0].v[:, :1]
    case[0].x[:, :60] = case[0].x[:, :1]
    _check(ctx, vr, ref, case, 32, 8)


def test_subset_across_hosts(ctx, vr, ref):
    """A sparse subset: a wavefront's queries lie in many hosts and leaves."""
    rng = np.random.default_rng(8)
    case = _hosts(rng, [300] * 40 + [3000])
    sub = np.sort(rng.permutation(case[0].n)[:700]).astype(np.int32)
    _check(ctx, vr, ref, case, 32, 8, subset=rng.permutation(sub).astype(np.int32))


@pytest.mark.parametrize("n_se,n_v", [(32, 8), (256, 32)])
def test_host_wider_than_half_the_box(ctx, vr, ref, n_se, n_v):
    """0.7 of the box on every axis about the first member: no neighbour is
    nearer through the box, so plain differences give the periodic sets."""
    rng = np.random.default_rng(9)
    case = _hosts(rng, [6000, 700])
    x = 0.5 + 0.35 * (2 * rng.random((3, 6000)) - 1)
    x[:, 0] = 0.5
    case[0].x[:, :6000] = x
    _check(ctx, vr, ref, case, n_se, n_v)


@pytest.mark.parametrize("n_se,n_v", [(32, 8), (32, 32), (48, 16), (256, 32)])
def test_infinite_velocities(ctx, vr, ref, n_se, n_v):
    """R of the members of finite velocity where enough of the neighbours have
    one, and no number where too few do."""
    rng = np.random.default_rng(8)
    w, off, mem, vbar, sigma = _hosts(rng, [600, 600])
    few = rng.permutation(600)
    w.v[0, few[:60]] = np.inf
    w.v[1, 600 + few[4:]] = -np.inf
    P, Pr = both(ctx, vr, ref, w)
    exp = ref.local_vdensity(Pr, off, mem, vbar, sigma, n_se, n_v)["R"]
    got = ctx.local_vdensity(P, dev_tensor(off), dev_tensor(mem), dev_tensor(vbar), dev_tensor(sigma), n_se, n_v)
    fin = np.isfinite(w.v).all(axis=0)
    got = got.cpu().numpy()
    assert np.isnan(got[600:][fin[600:]]).all() and np.isnan(exp[600:][fin[600:]]).all()
    some = fin & (np.arange(1200) < 600)
    assert np.isfinite(exp[some]).any()
    R_agrees(got, exp, where=some)


@pytest.mark.parametrize("n_hosts,extent", [(1, 0.0), (1, 0.01), (300, 1e-4), (1024, 0.02), (2100, 0.08)])
def test_presort_key_widths(ctx, vr, ref, n_hosts, extent):
    """Keys relative to a host's box, of 1 to 32 bits and of more; hosts of
    coincident members and across the box's edge."""
    rng = np.random.default_rng(n_hosts)
    sizes = (64 + rng.integers(0, 40, n_hosts)).tolist() if n_hosts > 1 else [3000]
    _check(ctx, vr, ref, _hosts(rng, sizes, extent=extent), 32, 8)


@pytest.mark.parametrize("n_se,n_v,lo,hi", [(2, 2, 2, 5), (32, 8, 32, 70), (48, 16, 48, 130), (256, 32, 256, 300)])
@pytest.mark.parametrize("leaf", [16, 256])
def test_many_small_hosts(ctx, vr, ref, leaf, n_se, n_v, lo, hi):
    """More small buckets than the chip holds at once: a wavefront takes as many
    of them as 16 leaves hold, with larger ones and full ones in between."""
    rng = np.random.default_rng(n_se + leaf)
    sizes = rng.integers(lo, hi + 1, 900)
    sizes[[0, 100, 101, 450, 899]] = [512, 513, 511, 2500, 481]
    saved = ctx.get_tune("knn_leaf")
    try:
        ctx.tune("knn_leaf", leaf)
        _check(ctx, vr, ref, _hosts(rng, sizes.tolist(), extent=1e-3, masses=n_se == 48), n_se, n_v)
    finally:
        ctx.tune("knn_leaf", saved)


@pytest.mark.parametrize("n_hosts,size,n_se,n_v,subset,room", [(20000, 2, 2, 2, False, 360), (20000, 2, 2, 2, True, 372),
                                                               (3000, 33, 32, 8, False, 196), (3000, 33, 32, 8, True, 207),
                                                               (3000, 65, 32, 8, False, 190)])
def test_small_hosts_within_a_workspace_cap(vr, ref, n_hosts, size, n_se, n_v, subset, room):
    """Hosts that pad their leaves most, in as many ranges as `room` bytes a
    member allow (what the search needed before its leaves were padded)."""
    rng = np.random.default_rng(size)
    case = _hosts(rng, [size] * n_hosts, extent=1e-3)
    n = case[0].n
    capped = vr.Context(0, max_workspace_bytes=room * n)
    _check(capped, vr, ref, case, n_se, n_v, subset=rng.permutation(n)[:n // 2].astype(np.int32) if subset else None)
    assert capped.workspace_bytes() <= room * n


def test_ranges_of_hosts_of_all_sizes(vr, ref):
    """Large hosts between runs of small ones, whole and by a subset that leaves
    whole ranges out."""
    rng = np.random.default_rng(12)
    sizes = np.concatenate([rng.integers(32, 40, 2500), [5000], rng.integers(32, 40, 2500), [700, 4096], [33] * 300])
    case = _hosts(rng, sizes.tolist(), extent=2e-3, masses=True)
    n = case[0].n
    capped = vr.Context(0, max_workspace_bytes=215 * n)
    _check(capped, vr, ref, case, 32, 8)
    off = case[1]
    for lo, hi in ((0, n), (2490, 2510), (off[2500], off[2501]), (off[5001], n)):
        sub = rng.permutation(np.arange(lo, hi))[:1500].astype(np.int32)
        _check(capped, vr, ref, case, 32, 8, subset=sub)
