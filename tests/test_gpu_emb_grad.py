"""Embedding gradient and column sums in the launch of the FP32 weight gradients:
contexts whose (row, position) pairs end inside a step of 32, rows wider than a
sub-batch, and row counts around its chunks; and the same sums as launches of
their own (BF16 products).  Against the oracle: FP32 sums over up to 700 rows of
terms exact to 2^-24, 1e-4 of the tensor's largest; BF16 products 3e-2."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.model import Model as OModel

from .gpu_util import banner, lib_cfg, oracle_cfg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("precision,rtol", [("fp32", 1e-4), ("bf16", 3e-2)])
@pytest.mark.parametrize("context,embed,rows", [(4, 16, 1), (4, 64, 130), (20, 32, 17), (100, 16, 7), (12, 16, 700),
                                                (256, 64, 3), (256, 32, 65)])
def test_gradients(E, precision, rtol, context, embed, rows):
    model = dict(context=context, embed=embed, latent=16, blocks=1, hidden=16, branches=2, lr=1e-3,
                 beta1=0.9, beta2=0.999, eps=1e-8, seed=5)
    rng = np.random.RandomState(context + rows)
    ctx = rng.randint(0, 256, (rows, context)).astype(np.uint8)
    tgt = rng.randint(0, 256, rows).astype(np.uint8)
    slots = rng.permutation(rows)
    d_ctx, d_tgt = (torch.as_tensor(a).to("cuda") for a in (ctx, tgt))
    banner(f"embedding gradient C {context} E {embed} rows {rows} {precision}")
    m = E.Model(lib_cfg(E, model, precision), rows, rows)
    m.edpc_model_step(d_ctx, d_tgt, slots, flags=E.EDPC_STEP_BACKWARD)
    om = OModel(oracle_cfg(model), rows)
    g_o, _ = om.backward(om.forward(ctx.astype(np.int64), slots), tgt.astype(np.int64))
    for n in ("emb", "b1", "b2", "bh"):
        g = m.edpc_model_read(n, E.EDPC_KIND_GRAD)
        assert np.abs(g - g_o[n].reshape(-1)).max() <= rtol * np.abs(g_o[n]).max(), n
