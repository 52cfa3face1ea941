"""FP32 row-block kernel at the upper end of its rows: up to 4095 it repeats the
layer-by-layer launches bit for bit, 4096 rows leave it, and so do fewer rows of a model
made for 4096 (whose LayerNorm adjoint forms column sums)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

MODEL = dict(context=16, embed=16, latent=64, blocks=1, hidden=64, branches=2, lr=1e-3, beta1=0.9, beta2=0.999,
             eps=1e-8, seed=8)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("branches", [1, 2, 3])
@pytest.mark.parametrize("rows,most", [(1000, 1000), (4081, 4095), (4095, 4095), (4095, 4096), (4096, 4096)])
def test_rows(E, rows, most, branches):
    rng = np.random.RandomState(rows)
    banner(f"FP32 row block {rows} of {most} rows, {branches} branches")
    ms = [E.Model(lib_cfg(E, dict(MODEL, branches=branches), layerwise=lw), most, most) for lw in (False, True)]
    for flags in (E.EDPC_STEP_BACKWARD, E.EDPC_STEP_UPDATE, 0):
        ctx = torch.as_tensor(rng.randint(0, 256, (rows, 16)).astype(np.uint8)).to("cuda")
        tgt = torch.as_tensor(rng.randint(0, 256, rows).astype(np.uint8)).to("cuda")
        slots = rng.permutation(most)[:rows]
        out = []
        for m in ms:
            p, loss = torch.empty(rows, 256, device="cuda"), torch.empty(1, device="cuda")
            m.edpc_model_step(ctx, tgt, slots, probs=p, loss=loss, flags=flags)
            out.append([p.cpu().numpy(), loss.cpu().numpy()] + [m.edpc_model_read(n) for n in m.names] +
                       [m.edpc_model_read(n, E.EDPC_KIND_GRAD) for n in m.names if flags and n != "U"])
        for i, (a, b) in enumerate(zip(*out)):
            assert np.array_equal(a, b), (flags, i)
