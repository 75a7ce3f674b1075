"""R in hosts of half the box's width or more, where a neighbour may be nearer
through the box than by the coordinates unwrapped about the first member: the
periodic sets of the oracle, whatever the buckets and whichever other hosts the
call holds."""
import numpy as np
import pytest

from paper_1902_01010_amd import pipeline, synth
from tests.gpu_common import R_agrees, both, dev_tensor
from tests.test_gpu_knn import _check, _hosts

pytestmark = pytest.mark.gpu

BITS = 21


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


def _filled(rng, n, axes, narrow=(), masses=False):
    """A host that fills the box along `axes` (0.2 of it along the others),
    with a dense clump across the unwrapped edge, and Gaussian narrow hosts."""
    case = _hosts(rng, [n, *narrow], masses=masses)
    x = 0.4 + 0.2 * rng.random((3, n))
    x[:, 1:n // 4] = 0.5 + 0.01 * rng.normal(size=(3, n // 4 - 1))
    for a in axes:
        x[a, n // 4:] = rng.random(n - n // 4)
        x[a, 1:n // 4] += 0.25  # the clump about 0.75,
        x[a, 0] = 0.25          # where the unwrapped edge is
    case[0].x[:, :n] = np.mod(x, 1).astype(np.float32)
    case[0].x[case[0].x >= 1] = 0
    return case


@pytest.mark.parametrize("n_se,n_v", [(2, 2), (32, 8), (48, 16), (100, 20), (256, 32)])
@pytest.mark.parametrize("axes", [(0,), (2,), (0, 1, 2)])
def test_sets_across_the_unwrapped_edge(ctx, vr, ref, axes, n_se, n_v):
    """A wide host between narrow ones; R does not depend on the buckets."""
    rng = np.random.default_rng(n_se + 7 * len(axes))
    case = _filled(rng, 3000, axes, narrow=[600, 257], masses=n_se == 48)
    saved = ctx.get_tune("knn_leaf")
    try:
        for leaf in (16, 64, 256):
            ctx.tune("knn_leaf", leaf)
            _check(ctx, vr, ref, case, n_se, n_v)
    finally:
        ctx.tune("knn_leaf", saved)


def test_subset_of_a_wide_host(ctx, vr, ref):
    rng = np.random.default_rng(4)
    case = _filled(rng, 4000, (0, 1, 2), narrow=[700])
    _check(ctx, vr, ref, case, 32, 8, subset=rng.permutation(case[0].n)[:500].astype(np.int32))


@pytest.mark.parametrize("n_se,n_v", [(32, 8), (48, 16), (100, 20), (256, 32)])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("delta", [-1, 0, 1])
@pytest.mark.parametrize("low", [False, True])
def test_one_grid_unit_round_the_reach_of_a_set(ctx, vr, ref, low, delta, axis, n_se, n_v):
    """A query at one unwrapped end whose n_se-th neighbour on its side is r
    away and a member of the other end r + delta through the box: in the set
    below r, at r by its index, not beyond."""
    rng = np.random.default_rng(10 * n_se + axis)
    r, full, q0 = 2 * n_se, 1 << BITS, 7
    other = (axis + 1) % 3
    q = np.full((3, 400 + n_se), full // 2)
    q[:, 1:400] = full // 4 + rng.integers(0, full // 2, (3, 399))   # the host's bulk, about the first member
    near = q[:, 400:]
    near[axis] = q0
    near[other] += np.concatenate([np.arange(n_se - 1), [r]])        # the query at 400, n_se - 1 neighbours
    image = 1 if low else 399                                        # the other end's member, before or after them
    q[:, image] = near[:, 0]
    q[axis, image] = full + q0 - (r + delta)
    if not low:  # last of all
        q = np.concatenate([np.delete(q, image, axis=1), q[:, image:image + 1]], axis=1)
        image = q.shape[1] - 1
    n = q.shape[1]
    query = 400 if low else 399
    w, off, mem, vbar, sigma = _hosts(rng, [n])
    w.x[:] = q / full
    P, Pr = both(ctx, vr, ref, w)
    exp = ref.local_vdensity(Pr, off, mem, vbar, sigma, n_se, n_v, want_sets=True)
    assert (image in exp["nbr_s"][query]) == (delta < 0 or (delta == 0 and low))
    got = ctx.local_vdensity(P, dev_tensor(off), dev_tensor(mem), dev_tensor(vbar), dev_tensor(sigma), n_se, n_v)
    R_agrees(got.cpu().numpy(), exp["R"])


@pytest.mark.parametrize("seed", [3, 22])
def test_halo_that_spans_the_box(ctx, vr, ref, seed):
    """The isolated halo of 100,000 particles, for seeds whose host reaches
    round the box: R near its unwrapped ends."""
    w = synth.isolated_halo(seed=seed, n_host=100000, n_sub=5, sub_range=(5555, 5555))
    P, Pr = both(ctx, vr, ref, w)
    prm = pipeline.Params.from_workload(w)
    _, _, off, mem = ctx.groups(ctx.fof3d(P, prm.ellx), 256)
    off, mem = off[:2].contiguous(), mem[:int(off[1])].contiguous()
    cm = ctx.cell_moments(P, off, mem)
    got = ctx.local_vdensity(P, off, mem, cm["vbar"], cm["sigma"], 32, 8).cpu().numpy()
    m = mem.cpu().numpy()
    x = w.x[:, m].astype(np.float64)
    d = np.abs((x - x[:, :1] + 0.5 * w.box) % w.box - 0.5 * w.box).max(axis=0)
    ends = m[np.argsort(-d)[:1500]].astype(np.int32)
    exp = ref.local_vdensity(Pr, off.cpu().numpy(), m, np.ascontiguousarray(cm["vbar"].cpu().numpy()),
                             np.ascontiguousarray(cm["sigma"].cpu().numpy()), 32, 8, subset=ends)["R"]
    R_agrees(got[ends], exp[ends])
