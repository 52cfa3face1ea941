"""An explicit step captured by its caller, replayed several times with other inputs and
eager work between the replays: outputs and kept FDM gradients are those of the same
step launched directly, in and outside the slots of the call."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

MODEL = dict(context=16, embed=16, latent=64, blocks=2, hidden=128, branches=2, lr=1e-3, beta1=0.9, beta2=0.999,
             eps=1e-8, seed=3)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_kept_gradients(E, precision):
    rows, slots = 7, 12
    banner(f"captured step {precision}")
    rng = np.random.RandomState(0)
    m, ref = (E.Model(lib_cfg(E, MODEL, precision), slots, slots) for _ in range(2))
    new = lambda *s: torch.as_tensor(rng.randint(0, 256, s).astype(np.uint8)).to("cuda")
    ctx, tgt = new(rows, 16), new(rows)
    probs = [torch.empty(rows, 256, device="cuda") for _ in range(2)]
    at = np.array([11, 0, 5, 3, 9, 1, 6])
    flags = E.EDPC_STEP_BACKWARD | E.EDPC_STEP_KEEP_FDM_GRAD
    m.edpc_model_step(ctx, tgt, at, probs=probs[0], flags=flags)  # (makes the memory of the gradients)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.edpc_model_step(ctx, tgt, at, probs=probs[0], flags=flags)
    for replay in range(4):
        ctx.copy_(new(rows, 16))
        tgt.copy_(new(rows))
        for mod in (m, ref):  # eager work of the same models, with every slot: leaves gradients in all of them
            mod.edpc_model_step(new(slots, 16), new(slots), np.arange(slots), flags=flags)
        torch.cuda.synchronize()
        g.replay()
        ref.edpc_model_step(ctx, tgt, at, probs=probs[1], flags=flags)
        torch.cuda.synchronize()
        assert torch.equal(*probs), replay
        for n in m.names:
            assert np.array_equal(m.edpc_model_read(n, E.EDPC_KIND_GRAD), ref.edpc_model_read(n, E.EDPC_KIND_GRAD)), n
        kept = m.edpc_model_read("U", E.EDPC_KIND_GRAD).reshape(slots, -1)
        assert not kept[[s for s in range(slots) if s not in at]].any()
