"""Row-block update over the weight-gradient ids of both instructions, for both shapes of
the row-block step and rows around its chunks of 64: the gradients that the launch with
Adam leaves are those of the plain launch, bit for bit, and parameters and moments
follow the formula.  Every model here must be on the row-block path (bit 47 of its id)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.model import Model as OModel

from .gpu_util import banner, lib_cfg, oracle_cfg

pytestmark = pytest.mark.gpu

F32 = 2.0 ** -23
BASE = dict(embed=16, branches=2, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, seed=11)
MODELS = {"small1": dict(BASE, context=16, latent=64, blocks=1, hidden=128),
          "mid2": dict(BASE, context=32, latent=128, blocks=2, hidden=256)}
WGRAD = 10  # product slot of the weight gradients


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 193])
@pytest.mark.parametrize("tile", [0, 2, 3, 6])  # 16 x 16 x 32 up to 2, 32 x 32 x 16 from 3
@pytest.mark.parametrize("model", list(MODELS))
def test_update(E, model, tile, rows):
    cfg = MODELS[model]
    given = E.Model(lib_cfg(E, cfg, "bf16"), rows, rows).edpc_model_kernel_id()
    assert given >> 47 & 1, "left the row-block step"
    kid = given & ~(0xF << 4 * WGRAD) | tile << 4 * WGRAD
    rng = np.random.RandomState(rows + tile)
    d_ctx = torch.as_tensor(rng.randint(0, 256, (rows, cfg["context"])).astype(np.uint8)).to("cuda")
    d_tgt = torch.as_tensor(rng.randint(0, 256, rows).astype(np.uint8)).to("cuda")
    slots = rng.permutation(rows)
    banner(f"row-block update {model}, id {tile}, {rows} rows")
    m = E.Model(lib_cfg(E, cfg, "bf16"), rows, rows, kid)
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
    # written parameters rebuild both fragment copies: they must predict and differentiate alike
    m2 = E.Model(lib_cfg(E, cfg, "bf16"), rows, rows, kid)
    for n in names + ["U"]:
        m2.edpc_model_write(n, m.edpc_model_read(n))
    probs = [torch.empty(rows, 256, device="cuda") for _ in range(2)]
    for k, mod in enumerate((m, m2)):
        mod.edpc_model_step(d_ctx, d_tgt, slots, probs=probs[k], flags=E.EDPC_STEP_BACKWARD)
    assert torch.equal(*probs)
    for n in names:
        assert np.array_equal(m.edpc_model_read(n, E.EDPC_KIND_GRAD), m2.edpc_model_read(n, E.EDPC_KIND_GRAD)), n
