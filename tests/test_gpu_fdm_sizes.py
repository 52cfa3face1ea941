"""Feature Distribution Matrix kernels over the sizes where their split and
cache policy change: one to four workgroups a slot (L = 16 .. 256), and states
that are cached, stream their moments, or stream altogether (the last from
1025 slots of 256 x 256).  Gradients against the oracle (FP32 sums over
K <= 256: 1e-4 of the tensor's largest), and the Adam update of U_s against its
formula on the gradient that the library reports (FP32 rounding)."""

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


@pytest.mark.parametrize("latent,rows", [(16, 3), (32, 70), (64, 37), (128, 5), (128, 2600), (256, 3), (256, 1040)])
def test_gradients_and_update(E, latent, rows):
    model = dict(context=4, embed=16, latent=latent, blocks=1, hidden=16, branches=2, lr=1e-3,
                 beta1=0.9, beta2=0.999, eps=1e-8, seed=5)
    rng = np.random.RandomState(latent + rows)
    ctx, tgt = rng.randint(0, 256, (rows, 4)).astype(np.uint8), rng.randint(0, 256, rows).astype(np.uint8)
    slots = rng.permutation(rows)
    d_ctx, d_tgt = (torch.as_tensor(a).to("cuda") for a in (ctx, tgt))
    banner(f"FDM latent {latent}, {rows} rows")
    m = E.Model(lib_cfg(E, model), rows, rows)
    m.edpc_model_step(d_ctx, d_tgt, slots, flags=E.EDPC_STEP_BACKWARD | E.EDPC_STEP_KEEP_FDM_GRAD)
    dU = m.edpc_model_read("U", E.EDPC_KIND_GRAD)
    u0 = m.edpc_model_read("U").astype(np.float64)
    om = OModel(oracle_cfg(model), rows)
    c = om.forward(ctx.astype(np.int64), slots)
    g_o, dU_o = om.backward(c, tgt.astype(np.int64))
    got = dU.reshape(rows, latent, latent)[slots]
    assert np.abs(got - dU_o).max() <= 1e-4 * np.abs(dU_o).max()
    for n in ("emb", "w1", "b1"):  # what dx' = U_s dy feeds
        g = m.edpc_model_read(n, E.EDPC_KIND_GRAD)
        assert np.abs(g - g_o[n].reshape(-1)).max() <= 1e-4 * np.abs(g_o[n]).max(), n
    del om, c, g_o, dU_o, got
    m.edpc_model_step(d_ctx, d_tgt, slots, flags=E.EDPC_STEP_UPDATE)
    g = dU.astype(np.float64)
    b1, b2, lr, eps = (float(np.float32(x)) for x in (0.9, 0.999, 1e-3, 1e-8))
    mo, vo = (1 - b1) * g, (1 - b2) * g * g
    step = lr * (mo / (1 - b1)) / (np.sqrt(vo / (1 - b2)) + eps)
    assert np.all(np.abs(m.edpc_model_read("U", E.EDPC_KIND_ADAM_M) - mo) <= 4 * F32 * np.abs(g) + 1e-30)
    assert np.all(np.abs(m.edpc_model_read("U", E.EDPC_KIND_ADAM_V) - vo) <= 4 * F32 * g * g + 1e-30)
    assert np.all(np.abs(m.edpc_model_read("U") - (u0 - step))
                  <= F32 * (2 * np.abs(u0) + 16 * np.abs(step)) + 1e-12)
