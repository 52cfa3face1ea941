"""FP32 autotuner: products that the row-block kernel replaces keep their ids (another
instruction for one of them would take that kernel away), the others come out as the
default or as the one id of the other instruction, and a tuned model's steps are
those of a model given its id."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

BASE = dict(embed=16, branches=2, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, seed=9)
SMALL = dict(BASE, context=16, latent=64, blocks=2, hidden=128)
MID = dict(BASE, context=32, latent=128, blocks=2, hidden=256)
SLOTS = 11        # products of a step, 4 bits of the id each
DOWN, DOWN_BWD, WGRAD = 0, 9, 10
CLASS = (0, 3)    # 16 x 16 x 4 up to id 2, 32 x 32 x 2 from id 3 on


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("model,rows", [("small", 8), ("small", 1024), ("mid", 8), ("mid", 1024), ("mid", 4200)])
def test_ids(E, model, rows):
    cfg = SMALL if model == "small" else MID
    banner(f"FP32 autotuner {model} {rows} rows")
    given = E.Model(lib_cfg(E, cfg), rows, rows).edpc_model_kernel_id()
    m = E.Model(lib_cfg(E, cfg, autotune=True), rows, rows)
    tuned = m.edpc_model_kernel_id()
    assert given >> 44 == tuned >> 44
    for s in range(SLOTS):
        g, t = (k >> (4 * s) & 15 for k in (given, tuned))
        if s == WGRAD:
            assert t <= 6
        elif model == "small" and s not in (DOWN, DOWN_BWD):
            assert t == g, s
        else:
            assert t == g or t == CLASS[g < 3], (s, g, t)
    m2 = E.Model(lib_cfg(E, cfg), rows, rows, tuned)
    rng = np.random.RandomState(rows)
    for step in range(2):
        ctx = torch.as_tensor(rng.randint(0, 256, (rows, cfg["context"])).astype(np.uint8)).to("cuda")
        tgt = torch.as_tensor(rng.randint(0, 256, rows).astype(np.uint8)).to("cuda")
        probs = [torch.empty(rows, 256, device="cuda") for _ in range(2)]
        for mod, p in zip((m, m2), probs):
            mod.edpc_model_step(ctx, tgt, np.arange(rows), probs=p, flags=E.EDPC_STEP_UPDATE)
        assert torch.equal(*probs)
    for n in m.names:
        assert np.array_equal(m.edpc_model_read(n), m2.edpc_model_read(n)), n
