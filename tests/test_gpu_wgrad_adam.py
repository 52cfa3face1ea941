"""Row-block step: the launch that sums the weight gradients and applies Adam,
over both shapes (32 x 32 x 16 and 16 x 16 x 32 instructions) and row counts
around its chunks of 64.  The gradients it leaves are those of the plain
weight-gradient launch, bit for bit (the same instruction over ascending rows),
and parameters and moments follow the formula (FP32 rounding); the fragment
copies are seen through the next step's probabilities, against a model given
the same parameters."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.model import Model as OModel

from .gpu_util import banner, lib_cfg, oracle_cfg

pytestmark = pytest.mark.gpu

F32 = 2.0 ** -23
BASE = dict(embed=16, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, seed=11)
MODELS = {"small": dict(BASE, context=16, latent=64, blocks=2, hidden=128, branches=2),
          "mid": dict(BASE, context=32, latent=128, blocks=1, hidden=256, branches=2),
          "mid4": dict(BASE, context=32, latent=128, blocks=4, hidden=256, branches=2),
          "small1": dict(BASE, context=16, latent=64, blocks=1, hidden=128, branches=1)}


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("rows", [1, 63, 65, 128, 193, 449])
@pytest.mark.parametrize("model", list(MODELS))
def test_update(E, model, rows):
    cfg = MODELS[model]
    rng = np.random.RandomState(rows)
    ctx = rng.randint(0, 256, (rows, cfg["context"])).astype(np.uint8)
    tgt = rng.randint(0, 256, rows).astype(np.uint8)
    slots = rng.permutation(rows)
    d_ctx, d_tgt = (torch.as_tensor(a).to("cuda") for a in (ctx, tgt))
    banner(f"row-block update {model}, {rows} rows")
    m = E.Model(lib_cfg(E, cfg, "bf16"), rows, rows)
    names = list(OModel(oracle_cfg(cfg), 1).p)
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
    # writing parameters rebuilds the fragment copies: both must predict alike
    m2 = E.Model(lib_cfg(E, cfg, "bf16"), rows, rows)
    for n in names + ["U"]:
        m2.edpc_model_write(n, m.edpc_model_read(n))
    probs = [torch.empty(rows, 256, device="cuda") for _ in range(2)]
    for k, mod in enumerate((m, m2)):
        mod.edpc_model_step(d_ctx, d_tgt, slots, probs=probs[k], flags=E.EDPC_STEP_BACKWARD)
    assert torch.equal(*probs)
    for n in names:
        assert np.array_equal(m.edpc_model_read(n, E.EDPC_KIND_GRAD), m2.edpc_model_read(n, E.EDPC_KIND_GRAD)), n
