"""The 6D linker's tiles where they can go wrong: cells of one participant to
several tiles, around 64 (one wavefront or two a tile), the smallest tiled grid
(four cells a side, every neighbour across a face somewhere), several hosts in
one cell, components that most of a cell belongs to with some outside, and
velocity scales beyond the FP32 test's range.  Labels are exact, for both
linking criteria."""
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


def _clumps(counts, bits, side, seed, vscale):
    """Clumps of the given sizes, one a cell of `side`, the first across the
    box's corner; a third of each clump shares a velocity, the rest spread."""
    rng = np.random.default_rng(seed)
    nc = (1 << bits) // side
    q, v = [], []
    for i, m in enumerate(counts):
        c = np.array([i % nc, (i // nc) % nc, (i * 7) % nc])[:, None] * side
        q.append(c + (rng.integers(0, side, (3, m)) if i % 2 else np.rint(rng.normal(0, side / 4, (3, m))).astype(np.int64)))
        w = rng.normal(0, 1.0, (3, m))
        w[:, :m // 3] *= 0.05
        v.append(w * vscale)
    q = (np.concatenate(q, axis=1) % (1 << bits)).astype(np.uint32)
    return q, np.concatenate(v, axis=1).astype(np.float32)


@pytest.mark.parametrize("bits,side", [(21, 1 << 19), (21, 4096), (10, 64)])
@pytest.mark.parametrize("n_hosts", [1, 3])
@pytest.mark.parametrize("vscale", [1.0, 1e-17, 1e17])
def test_tiles(ctx, vr, ref, bits, side, n_hosts, vscale):
    counts = [1, 63, 64, 65, 127, 128, 129, 2, 300, 7, 1000, 5]
    q, v = _clumps(counts, bits, side, bits + n_hosts, vscale)
    n = q.shape[1]
    ell = 0.9 * side / (1 << bits)
    rng = np.random.default_rng(n_hosts)
    host = rng.integers(0, n_hosts, n).astype(np.int32)
    host[rng.random(n) < 0.02] = -1
    ellv = np.linspace(1.0, 1.3, n_hosts) * vscale
    P, Pr = vr.Particles(dev_tensor(q.view(np.int32)), dev_tensor(v), None, 1.0, 1.0, bits), ref.Particles(q, v, None, 1.0, 1.0, bits)
    exp = ref.fof6d(Pr, host, ellv, ell, None, 2.0)
    got = ctx.fof6d(P, dev_tensor(host), dev_tensor(ellv), ell, None, 2.0).cpu().numpy()
    assert (got == exp).all()
    if vscale == 1.0:
        vbar = rng.normal(0, 0.1, (n, 3)).astype(np.float32)
        L = rng.normal(2.5, 1.0, n).astype(np.float32)
        exp = ref.fof_sub(Pr, host, n_hosts, vbar.T, ell, L, 2.0, 2.0, theta_op=0.6)
        got = ctx.fof_sub(P, dev_tensor(host), n_hosts, dev_tensor(vbar).t(), ell, dev_tensor(L), 2.0, 2.0, theta_op=0.6)
        assert (got.cpu().numpy() == exp).all()
