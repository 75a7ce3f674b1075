"""The masked 3D link at the shapes where it can go wrong: fine grids of 1, 2
and 4 a coarse side, the smallest coarse grid (4 a side, every row wrapping),
fine cells of many particles just beyond each other's reach (listed pairs),
and clumps across the box faces.  Labels are bit-exact."""
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


def _labels(ctx, vr, ref, q, bits, ell_u):
    size = 1 << bits
    Pd = vr.Particles(dev_tensor(q.view(np.int32)), None, None, 1.0, 1.0, bits)
    Pr = ref.Particles(q, None, None, 1.0, 1.0, bits)
    exp = ref.fof3d(Pr, ell_u / size)
    assert (ctx.fof3d(Pd, ell_u / size).cpu().numpy() == exp).all()
    return exp


@pytest.mark.parametrize("bits,ell_u,scale", [(21, 1500.0, 3000.0), (21, 2000.0, 3000.0), (12, 0.9, 6.0), (12, 1.2, 6.0),
                                              (12, 2.9, 12.0), (10, 200.0, 60.0), (10, 255.9, 200.0), (12, 900.0, 700.0)])
@pytest.mark.parametrize("wrap", [False, True])
def test_grids_and_box_faces(ctx, vr, ref, bits, ell_u, scale, wrap):
    rng = np.random.default_rng(int(ell_u))
    size = 1 << bits
    pos = np.concatenate([rng.normal(0, scale, (3, 4000)), rng.normal(0, 5 * scale, (3, 3000)),
                          rng.uniform(0, size, (3, 1500))], axis=1) + (0.0 if wrap else size / 2)
    q = np.mod(np.rint(pos), size).astype(np.uint32)
    _labels(ctx, vr, ref, q, bits, ell_u)


@pytest.mark.parametrize("gap,joined", [(1498, True), (1501, False)])
def test_many_particles_at_the_reach(ctx, vr, ref, gap, joined):
    """Two clumps of 3,000 particles each in one fine cell, whose nearest pair
    lies `gap` apart on x: thousands of pairs to test, one of them (or none)
    within the linking length."""
    rng = np.random.default_rng(1)
    a = np.stack([rng.integers(0, 100, 3000), rng.integers(0, 40, 3000), rng.integers(0, 40, 3000)])
    b = np.stack([rng.integers(0, 100, 3000), rng.integers(0, 40, 3000), rng.integers(0, 40, 3000)])
    a[:, 7] = (99, 20, 20)
    b[:, 9] = (0, 20, 20)
    a[0, a[0] == 99] = 98
    b[0, b[0] == 0] = 1
    a[0, 7], b[0, 9] = 99, 0
    x0 = 100 * 2048
    q = np.concatenate([a, b + np.array([[99 + gap], [0], [0]])], axis=1).astype(np.int64) + x0
    lab = _labels(ctx, vr, ref, q.astype(np.uint32), 21, 1500.0)
    assert (lab[0] == lab[3000]) == joined


@pytest.mark.parametrize("bits,ell_u,scale", [(21, 1500.0, 3000.0), (12, 0.9, 6.0), (12, 2.9, 12.0), (10, 200.0, 60.0),
                                              (10, 255.9, 200.0), (12, 900.0, 700.0)])
@pytest.mark.parametrize("n", [32768, 32769])
def test_lane_per_cell_and_per_neighbour(ctx, vr, ref, bits, ell_u, scale, n):
    """The same shapes on both sides of the size from which on a lane takes all
    of a cell's neighbours."""
    rng = np.random.default_rng(n + int(ell_u))
    size = 1 << bits
    a, b = n // 2, n // 3
    pos = np.concatenate([rng.normal(0, scale, (3, a)), rng.normal(0, 5 * scale, (3, b)),
                          rng.uniform(0, size, (3, n - a - b))], axis=1)
    _labels(ctx, vr, ref, np.mod(np.rint(pos), size).astype(np.uint32), bits, ell_u)
