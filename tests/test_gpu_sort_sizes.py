"""Sorts and scans at the sizes where their form changes: one workgroup with
one or four pairs a thread, small and large tiles whose counts the scatter adds
up itself, and scanned counts; batched sorts of the three dimensions, with and
without a workspace cap; scans in one workgroup, with and without their tile
sums scanned; partitions with tiles of 256 and of 1,024 positions.  Labels, group lists and cell numbers are exact."""
import numpy as np
import pytest

from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu

BITS = 18


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


@pytest.fixture(scope="module")
def ctx(vr):
    return vr.Context(0)


def _clumps(n, seed):
    rng = np.random.default_rng(seed)
    k = max(2, n // 60)
    centre = rng.integers(0, 1 << BITS, (3, k))
    q = centre[:, rng.integers(0, k, n)] + np.rint(rng.normal(0, 40.0, (3, n))).astype(np.int64)
    return (q % (1 << BITS)).astype(np.uint32), rng.normal(0, 1.0, (3, n)).astype(np.float32)


@pytest.mark.parametrize("n", [2, 1023, 1024, 1025, 4096, 4097, 16384, 16385, 131072, 131073, 524288, 524289, 4200000])
def test_labels_and_groups(ctx, vr, ref, n):
    """Sorts of n 64-bit cell keys and up to n 32-bit labels, scans of n flags."""
    q, v = _clumps(n, n)
    P = vr.Particles(dev_tensor(q.view(np.int32)), None, None, 1.0, 1.0, BITS)
    exp = ref.fof3d(ref.Particles(q, None, None, 1.0, 1.0, BITS), 30.0 / (1 << BITS))
    lab = ctx.fof3d(P, 30.0 / (1 << BITS))
    assert (lab.cpu().numpy() == exp).all()
    ng, of, off, mem = ctx.groups(lab, 20)
    eng, eof, eoff, emem = ref.groups(exp, 20)
    assert ng == eng and (of.cpu().numpy() == eof).all() and (off.cpu().numpy() == eoff).all()
    assert (mem.cpu().numpy()[:emem.size] == emem).all()


@pytest.mark.parametrize("cap", [0, 1 << 32])
@pytest.mark.parametrize("n", [1000, 1024, 1025, 4097, 131073, 524288, 524289, 1048576, 1048577, 1050625])
def test_member_lists(vr, ref, n, cap):
    """One host of n members: three sorts of n keys each, and its tree's levels."""
    c = vr.Context(0, cap)
    q, v = _clumps(n, n + 1)
    P = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(v), None, 1.0, 1.0, BITS)
    off, mem = np.array([0, n], np.int32), np.arange(n, dtype=np.int32)
    exp = ref.cell_moments(ref.Particles(q, v, None, 1.0, 1.0, BITS), off, mem)
    got = c.cell_moments(P, dev_tensor(off), dev_tensor(mem))
    assert (got["cell_of"].cpu().numpy() == exp["cell_of"]).all()


@pytest.mark.parametrize("n", [1, 5, 4096, 131072, 131073])
@pytest.mark.parametrize("share", [0.0, 0.4, 1.0])
def test_groups_with_unlabelled(ctx, ref, n, share):
    """A share of unlabelled particles, which small sets sort with the rest."""
    rng = np.random.default_rng(n)
    lab = rng.integers(0, max(1, n // 30), n)
    lab[rng.random(n) < share] = -1
    _, first, inv = np.unique(lab, return_index=True, return_inverse=True)
    lab = np.where(lab < 0, -1, first[inv]).astype(np.int32)  # labels are smallest members
    ng, of, off, mem = ctx.groups(dev_tensor(lab), 20)
    eng, eof, eoff, emem = ref.groups(lab, 20)
    assert ng == eng and (of.cpu().numpy() == eof).all() and (off.cpu().numpy() == eoff).all()
    assert (mem.cpu().numpy()[:emem.size] == emem).all()


@pytest.mark.parametrize("n", [5000, 131072])
def test_labels_under_a_cap(vr, ref, n):
    """With a workspace cap the cells' counts are waited for as in large sets."""
    c = vr.Context(0, 1 << 30)
    q, v = _clumps(n, n)
    P = vr.Particles(dev_tensor(q.view(np.int32)), None, None, 1.0, 1.0, BITS)
    exp = ref.fof3d(ref.Particles(q, None, None, 1.0, 1.0, BITS), 30.0 / (1 << BITS))
    assert (c.fof3d(P, 30.0 / (1 << BITS)).cpu().numpy() == exp).all()
