"""FP32 row-block kernel against the layer-by-layer launches, which it repeats bit
for bit: probabilities, CDFs, losses, every gradient, and the state after updates,
over its shapes, numbers of branches and blocks, and rows around its groups of 16;
and coding through it, both ways."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.model import Model as OModel

from .gpu_util import banner, lib_cfg, oracle_cfg

pytestmark = pytest.mark.gpu

BASE = dict(context=16, embed=16, lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, seed=7)
SHAPES = [(64, 128, 2, 2), (64, 64, 1, 1), (128, 128, 3, 3), (256, 64, 2, 1), (64, 128, 2, 0)]  # L, H, branches, blocks


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("rows", [1, 16, 17, 333])
@pytest.mark.parametrize("latent,hidden,branches,blocks", SHAPES)
def test_steps(E, latent, hidden, branches, blocks, rows):
    cfg = dict(BASE, latent=latent, hidden=hidden, branches=branches, blocks=blocks)
    rng = np.random.RandomState(rows + latent)
    names = list(OModel(oracle_cfg(cfg), 1).p)
    banner(f"FP32 row block L {latent} H {hidden} k {branches} n {blocks} rows {rows}")
    ms = [E.Model(lib_cfg(E, cfg, layerwise=lw), rows + 3, rows) for lw in (False, True)]
    for flags in (0, E.EDPC_STEP_BACKWARD, E.EDPC_STEP_UPDATE, E.EDPC_STEP_UPDATE, E.EDPC_STEP_BACKWARD):
        ctx = torch.as_tensor(rng.randint(0, 256, (rows, 16)).astype(np.uint8)).to("cuda")
        tgt = torch.as_tensor(rng.randint(0, 256, rows).astype(np.uint8)).to("cuda")
        slots = rng.permutation(rows + 3)[:rows]
        out = []
        for m in ms:
            p, c, loss = (torch.empty(rows, 256, device="cuda"), torch.empty(rows, 257, dtype=torch.int32, device="cuda"),
                          torch.empty(1, device="cuda"))
            m.edpc_model_step(ctx, tgt, slots, probs=p, cum=c, loss=loss, flags=flags)
            r = [p.cpu().numpy(), c.cpu().numpy(), loss.cpu().numpy()]
            r += [m.edpc_model_read(n, E.EDPC_KIND_GRAD) for n in names if flags]
            r += [m.edpc_model_read(n) for n in names + ["U"]]
            out.append(r)
        for i, (a, b) in enumerate(zip(*out)):
            assert np.array_equal(a, b), (flags, i)
    act = [torch.empty(rows * 256, device="cuda") for _ in ms]
    for j in range(blocks + 1):
        for m, a in zip(ms, act):
            m.edpc_model_activation(j, a)
        assert torch.equal(*act), j


@pytest.mark.parametrize("lens", [[90], [60, 17, 16, 0, 80] * 7])
def test_coding(E, lens):
    cfg = dict(BASE, latent=64, hidden=128, branches=2, blocks=2)
    data = torch.as_tensor(np.random.RandomState(len(lens)).randint(97, 105, sum(lens)).astype(np.uint8)).to("cuda")
    banner(f"FP32 row block coding {len(lens)} streams")
    conts = [E.edpc_encode(lib_cfg(E, cfg, layerwise=lw), data, lens) for lw in (False, True)]
    head = 92 + 20 * len(lens) + 4
    assert torch.equal(conts[0][head:], conts[1][head:])
    for c in conts:
        assert torch.equal(E.edpc_decode(c)[0], data)
