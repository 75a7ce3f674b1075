"""Calls under the smallest workspace cap that each has run with: the result of
a context without a cap, within the room."""
import numpy as np
import pytest
import torch

from paper_1902_01010_amd import synth
from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vr():
    from paper_1902_01010_amd import vr as m
    return m


def _sparse(vr, ctx, n):
    """Particles mostly in grid cells of their own, the most cells there can be."""
    rng = np.random.default_rng(1)
    x = (rng.random((3, n)) * (1 - 1e-6)).astype(np.float32)
    v = rng.normal(0, 100, (3, n)).astype(np.float32)
    return rng, vr.Particles(ctx.quantize(dev_tensor(x), 1.0, 21), dev_tensor(v), None, 1.0, 1.0, 21)


def fof3d(vr, ctx, n):
    _, P = _sparse(vr, ctx, n)
    return [ctx.fof3d(P, 0.5 * n ** (-1 / 3))]


def fof3d_dm(vr, ctx, n):
    rng, P = _sparse(vr, ctx, n)
    return [ctx.fof3d_dm(P, 0.5 * n ** (-1 / 3), dev_tensor((rng.random(n) < 0.4).astype(np.uint8)))]


def _hosted(vr, ctx, n):
    rng, P = _sparse(vr, ctx, n)
    return rng, P, dev_tensor((np.arange(n) * 50 // n).astype(np.int32))


def fof6d(vr, ctx, n):
    rng, P, host = _hosted(vr, ctx, n)
    return [ctx.fof6d(P, host, dev_tensor(np.full(50, 100.0)), 0.5 * n ** (-1 / 3), None)]


def fof6d_outliers(vr, ctx, n):
    rng, P, host = _hosted(vr, ctx, n)
    R = dev_tensor(rng.normal(1.5, 1, n).astype(np.float32))
    return [ctx.fof6d(P, host, dev_tensor(np.full(50, 100.0)), 0.5 * n ** (-1 / 3), R, 1.0)]


def fof_sub(vr, ctx, n):
    rng, P, host = _hosted(vr, ctx, n)
    L = dev_tensor(rng.normal(1.5, 1, n).astype(np.float32))
    vbar = dev_tensor(rng.normal(0, 10, (3, n)).astype(np.float32))
    return [ctx.fof_sub(P, host, 50, vbar, 0.5 * n ** (-1 / 3), L, 1.0)]


def groups(vr, ctx, n):
    """Half of the particles carry a label."""
    i = np.arange(n)
    _, of, off, mem = ctx.groups(dev_tensor(np.where(i < n // 2, i // 40, -1).astype(np.int32)), 20)
    return [of, off, mem[:int(off[-1])]]


def assign_baryons(vr, ctx, n):
    rng, P, host = _hosted(vr, ctx, n)
    off = dev_tensor(np.searchsorted(host.cpu().numpy(), np.arange(51)).astype(np.int32))
    star = dev_tensor((rng.random(n) < 0.4).astype(np.uint8))
    out, _ = ctx.assign_baryons(P, off, dev_tensor(np.arange(n, dtype=np.int32)), star, host, n ** (-1 / 3), 100.0)
    return [out]


def unbind(vr, ctx, n):
    """Equal masses, persistent passes."""
    _, P = _sparse(vr, ctx, n)
    off = dev_tensor(np.linspace(0, n, 101).astype(np.int32))
    ub = ctx.unbind(P, off, dev_tensor(np.arange(n, dtype=np.int32)), 1e-3, 1e-3)
    return [ub["bound"], ub["phi"], ub["iters"]]


def train(vr, ctx, n):
    rng = np.random.default_rng(3)
    feat = dev_tensor(rng.normal(size=(n, 12)).astype(np.float32)).bfloat16().view(torch.int16)
    w = dev_tensor(synth.mlp_init(1))
    return list(ctx.mlp_grad(w, feat, dev_tensor(rng.normal(size=n).astype(np.float32))))


CALLS = {f.__name__: f for f in (
    fof3d, fof3d_dm, fof6d, fof6d_outliers, fof_sub, groups, assign_baryons, unbind, train)}

# (call, particles, bytes)
ROOM = [("fof3d", 20000, 2079011), ("fof3d", 200000, 19994736), ("fof3d_dm", 20000, 2569251),
        ("fof3d_dm", 200000, 23420408), ("fof6d", 20000, 3297780), ("fof6d", 200000, 34597218),
        ("fof6d_outliers", 20000, 2556727), ("fof6d_outliers", 200000, 23265044), ("fof_sub", 20000, 3128095),
        ("fof_sub", 200000, 28811670), ("groups", 100000, 4492281), ("assign_baryons", 20000, 1619863),
        ("assign_baryons", 200000, 15100764), ("unbind", 20000, 1353420), ("unbind", 200000, 12886565),
        ("train", 2048, 637609), ("train", 8192, 2407613), ("train", 20000, 5837002)]


@pytest.mark.parametrize("name,n,room", ROOM)
def test_same_result_within_the_cap(vr, name, n, room):
    call = CALLS[name]
    free = call(vr, vr.Context(0), n)
    capped = vr.Context(0, max_workspace_bytes=room)
    got = call(vr, capped, n)
    assert capped.workspace_bytes() <= room
    for a, b in zip(free, got):
        a, b = a.cpu().numpy(), b.cpu().numpy()
        if a.dtype.kind == "f":
            np.testing.assert_allclose(b, a, rtol=1e-5, atol=1e-6 * np.nanmax(np.abs(a)))
        else:
            assert (a == b).all()


@pytest.mark.parametrize("n", [131073, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("name", ["fof3d", "fof3d_dm", "fof6d", "groups"])
def test_same_result_with_counts_bounded_and_read(vr, name, n):
    """The buffers sized for a cell, run and group a particle against those
    sized for the counts read, which any cap asks for."""
    for a, b in zip(CALLS[name](vr, vr.Context(0), n), CALLS[name](vr, vr.Context(0, max_workspace_bytes=1 << 30), n)):
        assert torch.equal(a, b)
