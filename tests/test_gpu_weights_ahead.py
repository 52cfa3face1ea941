"""BF16 row-block kernel with and without the workgroups that read weights ahead
(up to 192 row blocks have them: 3072 rows).  They only read: a row's
probabilities do not depend on how many rows there are, and are the same bits."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

BASE = dict(embed=16, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, seed=2, blocks=2, branches=2)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("flags", ["none", "backward"])
@pytest.mark.parametrize("context,latent,hidden", [(16, 64, 128), (32, 128, 256)])
def test_rows_alike(E, context, latent, hidden, flags):
    cfg = dict(BASE, context=context, latent=latent, hidden=hidden)
    n = 3073
    rng = np.random.RandomState(context)
    ctx = torch.as_tensor(rng.randint(0, 256, (n, context)).astype(np.uint8)).to("cuda")
    tgt = torch.as_tensor(rng.randint(0, 256, n).astype(np.uint8)).to("cuda")
    fl = E.EDPC_STEP_BACKWARD if flags == "backward" else 0
    out = {}
    for rows in (17, 3072, 3073):
        banner(f"weights ahead F {16 * context} rows {rows} {flags}")
        m = E.Model(lib_cfg(E, cfg, "bf16"), n, rows)
        p = torch.empty(rows, 256, device="cuda")
        m.edpc_model_step(ctx[:rows].contiguous(), tgt[:rows].contiguous(), np.arange(rows), probs=p, flags=fl)
        out[rows] = p
    assert torch.equal(out[3073][:3072], out[3072]) and torch.equal(out[3072][:17], out[17])
