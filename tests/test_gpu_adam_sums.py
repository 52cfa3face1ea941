"""Gradients that Adam sums itself (biases, LayerNorm, embedding) in the
layer-by-layer update, with tensors that end inside a wave's 64 elements: the
gradients left by an update are those of a backward pass alone, bit for bit, and
parameters and moments follow the formula (FP32 rounding)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.model import Model as OModel

from .gpu_util import banner, lib_cfg, oracle_cfg

pytestmark = pytest.mark.gpu

F32 = 2.0 ** -23


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("hidden,embed,rows", [(16, 16, 1), (48, 32, 64), (80, 64, 65), (16, 16, 700)])
def test_update_gradients(E, precision, hidden, embed, rows):
    model = dict(context=4, embed=embed, latent=16, blocks=2, hidden=hidden, branches=2, lr=1e-3,
                 beta1=0.9, beta2=0.999, eps=1e-8, seed=11)
    rng = np.random.RandomState(rows + hidden)
    ctx, tgt = rng.randint(0, 256, (rows, 4)).astype(np.uint8), rng.randint(0, 256, rows).astype(np.uint8)
    slots = rng.permutation(rows)
    d_ctx, d_tgt = (torch.as_tensor(a).to("cuda") for a in (ctx, tgt))
    banner(f"Adam sums H {hidden} E {embed} rows {rows} {precision}")
    m = E.Model(lib_cfg(E, model, precision), rows, rows)
    names = list(OModel(oracle_cfg(model), 1).p)
    m.edpc_model_step(d_ctx, d_tgt, slots, flags=E.EDPC_STEP_BACKWARD)
    g0 = {n: m.edpc_model_read(n, E.EDPC_KIND_GRAD) for n in names}
    p0 = {n: m.edpc_model_read(n).astype(np.float64) for n in names}
    m.edpc_model_step(d_ctx, d_tgt, slots, flags=E.EDPC_STEP_UPDATE)
    b1, b2, lr, eps = (float(np.float32(x)) for x in (0.9, 0.999, 1e-3, 1e-8))
    for n in names:
        assert np.array_equal(m.edpc_model_read(n, E.EDPC_KIND_GRAD), g0[n]), n
        g = g0[n].astype(np.float64)
        mo, vo = (1 - b1) * g, (1 - b2) * g * g
        step = lr * (mo / (1 - b1)) / (np.sqrt(vo / (1 - b2)) + eps)
        assert np.all(np.abs(m.edpc_model_read(n, E.EDPC_KIND_ADAM_M) - mo) <= 4 * F32 * np.abs(g) + 1e-30), n
        assert np.all(np.abs(m.edpc_model_read(n, E.EDPC_KIND_ADAM_V) - vo) <= 4 * F32 * g * g + 1e-30), n
        assert np.all(np.abs(m.edpc_model_read(n) - (p0[n] - step))
                      <= F32 * (2 * np.abs(p0[n]) + 16 * np.abs(step)) + 1e-12), n
