"""How a step gets its inputs: explicit steps around the number of rows whose
slots travel as kernel arguments (768), and coding steps of the shortest and
longest contexts, whose first kernel gathers and embeds.  Probabilities against
the oracle (FP32 logits of magnitude about 1, sums over K <= 64: 1e-5)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.codec import split_streams
from oracle.model import Model as OModel
from oracle.rangecoder import RangeEncoder

from .gpu_util import banner, lib_cfg, oracle_cfg, parse_container

pytestmark = pytest.mark.gpu

TINY = dict(context=4, embed=16, latent=16, blocks=1, hidden=16, branches=2, lr=1e-3, beta1=0.9,
            beta2=0.999, eps=1e-8, seed=3)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("rows", [1, 63, 257, 767, 768, 769])
def test_explicit_rows(E, rows):
    rng = np.random.RandomState(rows)
    n = 800
    ctx, tgt = rng.randint(0, 256, (rows, 4)).astype(np.uint8), rng.randint(0, 256, rows).astype(np.uint8)
    slots = rng.permutation(n)[:rows]
    d_ctx, d_tgt = (torch.as_tensor(a).to("cuda") for a in (ctx, tgt))
    banner(f"explicit step, {rows} rows")
    m, om = E.Model(lib_cfg(E, TINY), n, rows), OModel(oracle_cfg(TINY), n)
    p = torch.empty(rows, 256, device="cuda")
    m.edpc_model_step(d_ctx, None, slots, probs=p)
    c = om.forward(ctx.astype(np.int64), slots)
    assert np.abs(p.cpu().numpy() - c["p"]).max() <= 1e-5
    m.edpc_model_step(d_ctx, d_tgt, slots, flags=E.EDPC_STEP_BACKWARD)
    g_o, _ = om.backward(c, tgt.astype(np.int64))
    for name in ("emb", "w1"):  # the targets arrived
        g = m.edpc_model_read(name, E.EDPC_KIND_GRAD)
        assert np.abs(g - g_o[name].reshape(-1)).max() <= 1e-4 * np.abs(g_o[name]).max()


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("context,lens", [(4, [30, 4, 5, 0, 1, 29, 30]), (256, [300, 256, 257, 0, 299, 7])])
def test_coding_context_lengths(E, precision, context, lens):
    # the payloads of a coding call are those of the oracle's coder on the tables
    # of explicit steps over the same rows (longest stream first), byte for byte
    cfg, n = dict(TINY, context=context), len(lens)
    rng = np.random.RandomState(context)
    data = rng.randint(97, 105, sum(lens)).astype(np.uint8)
    banner(f"coding, context {context} {precision}")
    cont = E.edpc_encode(lib_cfg(E, cfg, precision), torch.as_tensor(data).to("cuda"), lens)
    out, lens_back = E.edpc_decode(cont)
    assert list(lens_back) == lens and out.cpu().numpy().tobytes() == data.tobytes()
    _, pays = parse_container(cont.cpu().numpy().tobytes())
    st = split_streams(data, lens)
    m = E.Model(lib_cfg(E, cfg, precision), n, n)
    coders = [RangeEncoder(16) for _ in st]
    order = sorted(range(n), key=lambda s: -lens[s])
    for i in range(max(lens)):
        act = [s for s in order if lens[s] > i]
        if i < context:
            for s in act:
                coders[s].encode(256 * st[s][i], 256)
            continue
        ctx = np.stack([np.frombuffer(st[s][i - context:i], np.uint8) for s in act])
        tgt = np.array([st[s][i] for s in act], np.uint8)
        cum = torch.empty(len(act), 257, dtype=torch.int32, device="cuda")
        m.edpc_model_step(torch.as_tensor(ctx).to("cuda"), torch.as_tensor(tgt).to("cuda"), act, cum=cum,
                          flags=E.EDPC_STEP_UPDATE)
        for s, row, x in zip(act, cum.cpu().numpy().astype(np.int64), tgt):
            coders[s].encode(int(row[x]), int(row[int(x) + 1] - row[x]))
    for s, p in enumerate(pays):
        assert p == (coders[s].finish() if lens[s] else b"")
