"""FP32 products on both sides of the line between 16 x 16 and 32 x 32 tiles (64 tiles
of 32 x 32: 256 rows for 256 outputs, 512 for 128; for a K of 512 and 1024 features 127
tiles): a row's results are the same bits on either."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

MODEL = dict(context=16, embed=16, latent=128, blocks=2, hidden=128, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, seed=6)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("context", [16, 32, 64])
@pytest.mark.parametrize("branches", [1, 2, 3])
def test_line(E, branches, context):
    rng = np.random.RandomState(branches)
    ctx = torch.as_tensor(rng.randint(0, 256, (1024, context)).astype(np.uint8)).to("cuda")
    tgt = torch.as_tensor(rng.randint(0, 256, 1024).astype(np.uint8)).to("cuda")
    m = E.Model(lib_cfg(E, dict(MODEL, branches=branches, context=context), layerwise=True), 1024, 1024)
    got = {}
    for rows in (64, 256, 257, 480, 512, 513, 1024):
        banner(f"FP32 tile line, context {context}, {branches} branches, {rows} rows")
        p = torch.empty(rows, 256, device="cuda")
        m.edpc_model_step(ctx[:rows], tgt[:rows], np.arange(rows), probs=p,
                          flags=E.EDPC_STEP_BACKWARD | E.EDPC_STEP_KEEP_FDM_GRAD)
        got[rows] = p[:64].cpu().numpy(), m.edpc_model_read("U", E.EDPC_KIND_GRAD).reshape(1024, -1)[:64]
    for rows, (p, du) in got.items():
        assert np.array_equal(p, got[64][0]), rows
        if rows in (256, 512, 1024):  # 1 / rows scales the adjoint: a power of two, so exactly
            assert np.array_equal(du * np.float32(rows // 64), got[64][1]), rows
