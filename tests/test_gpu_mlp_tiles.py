"""Gradient of the surrogate's network at the batch sizes where its tiles can go
wrong: one row, a tile of 32 less and more one, the most tiles that have a
workgroup each and one more (four wavefronts a workgroup, the last without a
tile), several tiles a wavefront; features that are not 8-byte aligned.  The
arithmetic model (BF16 operands, wide sums) differs by FP32 sums and by values
on a BF16 rounding boundary only: 5e-3 per parameter block."""
import numpy as np
import pytest
import torch

from oracle import surrogate as S
from tests.gpu_common import dev_tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1902_01010_amd import vr
    return vr.Context(0)


BLOCKS = np.cumsum([0, 768, 64, 4096, 64, 4096, 64, 64, 1])


@pytest.mark.parametrize("m", [1, 31, 32, 33, 16384, 16385, 16384 + 97, 40000])
@pytest.mark.parametrize("shift", [0, 1])
def test_gradient(ctx, m, shift):
    rng = np.random.default_rng(m)
    w = (rng.normal(size=S.MLP_PARAMS) * 0.2).astype(np.float32)
    bits = S.bf16_bits(rng.normal(size=(m, 12)))
    y = rng.normal(size=m)
    raw = np.zeros(m * 12 + shift, np.int16)
    raw[shift:] = bits.view(np.int16).reshape(-1)
    feat = dev_tensor(raw)[shift:].view(m, 12)
    loss_model, g_model = S.loss_and_grad(w, S.bf16_from_bits(bits), y, bf16=True)
    g, loss = ctx.mlp_grad(dev_tensor(w), feat, dev_tensor(y.astype(np.float32)))
    g = g.cpu().numpy().astype(np.float64)
    assert float(loss.item()) == pytest.approx(loss_model, rel=1e-4)
    for a, b in zip(BLOCKS[:-1], BLOCKS[1:]):
        assert np.linalg.norm(g[a:b] - g_model[a:b]) <= 5e-3 * np.linalg.norm(g_model[a:b]), (a, b)
    out = ctx.mlp_forward(dev_tensor(w), feat)
    aligned = ctx.mlp_forward(dev_tensor(w), dev_tensor(raw[shift:].copy()).view(m, 12))
    assert torch.equal(out, aligned)
