"""Explicit steps whose contexts and targets lie in host memory, pageable or pinned:
they are copied, as at any number of rows, and never read by a kernel."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

SMALL = dict(context=16, embed=16, latent=64, blocks=1, hidden=64, branches=2, lr=1e-3, beta1=0.9, beta2=0.999,
             eps=1e-8, seed=2)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("rows", [5, 768, 769])
@pytest.mark.parametrize("ctx_at,tgt_at", [("host", "host"), ("pinned", "pinned"), ("cuda", "host"), ("host", "cuda")])
def test_host_inputs(E, rows, ctx_at, tgt_at):
    rng = np.random.RandomState(rows)
    ctx = torch.as_tensor(rng.randint(0, 256, (rows, 16)).astype(np.uint8))
    tgt = torch.as_tensor(rng.randint(0, 256, rows).astype(np.uint8))
    put = {"host": lambda t: t, "pinned": lambda t: t.pin_memory(), "cuda": lambda t: t.cuda()}
    banner(f"inputs on {ctx_at} and {tgt_at}, {rows} rows")
    out = []
    for a, b in ((ctx.cuda(), tgt.cuda()), (put[ctx_at](ctx), put[tgt_at](tgt))):
        m = E.Model(lib_cfg(E, SMALL), rows, rows)
        p, loss = torch.empty(rows, 256, device="cuda"), torch.empty(1, device="cuda")
        m.edpc_model_step(a, b, np.arange(rows), probs=p, loss=loss, flags=E.EDPC_STEP_UPDATE)
        m.edpc_model_step(a, None, np.arange(rows), probs=p)
        torch.cuda.synchronize()
        out.append((p.cpu(), loss.cpu(), m.edpc_model_read("w1")))
    for x, y in zip(*out):
        assert np.array_equal(np.asarray(x), np.asarray(y))
