"""Entropy cells of a host whose first split spans more tiles than the
partition adds up one by one."""
import numpy as np
import pytest

from paper_1902_01010_amd import synth
from tests.gpu_common import both, dev_tensor

pytestmark = pytest.mark.gpu


def test_host_of_more_tiles_than_are_added_up(ref):
    """4.3 M members behind a host that ends inside a tile: the first level's
    counts are scanned, the second's added up."""
    from paper_1902_01010_amd import vr
    rng = np.random.default_rng(2)
    sizes = [5003, 4_300_000]
    n = sum(sizes)
    x = np.mod(0.5 + 0.1 * rng.normal(size=(3, n)) * np.array([[1.0], [0.7], [1.2]]), 1).astype(np.float32)
    x[x >= 1] = 0
    x[2, ::3] = x[2, 0]  # members with equal coordinates: order by index
    w = synth.Workload("large", x, rng.normal(0, 100, (3, n)).astype(np.float32), None, 1.0, 1.0, 21, {}, {})
    ctx = vr.Context(0)
    P, Pr = both(ctx, vr, ref, w)
    off, mem = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32), np.arange(n, dtype=np.int32)
    got = ctx.cell_moments(P, dev_tensor(off), dev_tensor(mem), f_cell=0.25, ncell_div=4)["cell_of"].cpu().numpy()
    exp = ref.cell_moments(Pr, off, mem, f_cell=0.25, ncell_div=4)["cell_of"]
    assert (got == exp).all()
