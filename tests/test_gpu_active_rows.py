"""Coding steps of the BF16 row-block sequence as their streams run out, across its
groups of 16 rows: payloads are the oracle's coder on the tables of explicit steps
over the streams that are left, byte for byte (the two set the step's rows in
different ways, and take the same kernels)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.codec import split_streams
from oracle.rangecoder import RangeEncoder

from .gpu_util import banner, lib_cfg, parse_container

pytestmark = pytest.mark.gpu

CFG = dict(context=16, embed=16, latent=64, blocks=1, hidden=128, branches=2, lr=1e-3, beta1=0.9,
           beta2=0.999, eps=1e-8, seed=4)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("lens", [[30] + [17] * 16 + [24] * 16 + [0, 5], [40] * 16 + [33] * 17 + [16]])
def test_rows_run_out(E, lens):
    n = len(lens)
    rng = np.random.RandomState(n)
    data = rng.randint(97, 105, sum(lens)).astype(np.uint8)
    banner(f"BF16 row block, {n} streams run out")
    cont = E.edpc_encode(lib_cfg(E, CFG, "bf16"), torch.as_tensor(data).to("cuda"), lens)
    out, _ = E.edpc_decode(cont)
    assert out.cpu().numpy().tobytes() == data.tobytes()
    _, pays = parse_container(cont.cpu().numpy().tobytes())
    st = split_streams(data, lens)
    m = E.Model(lib_cfg(E, CFG, "bf16"), n, n)
    coders = [RangeEncoder(16) for _ in st]
    order = sorted(range(n), key=lambda s: -lens[s])
    C = CFG["context"]
    for i in range(max(lens)):
        act = [s for s in order if lens[s] > i]
        if i < C:
            for s in act:
                coders[s].encode(256 * st[s][i], 256)
            continue
        ctx = np.stack([np.frombuffer(st[s][i - C:i], np.uint8) for s in act])
        tgt = np.array([st[s][i] for s in act], np.uint8)
        cum = torch.empty(len(act), 257, dtype=torch.int32, device="cuda")
        m.edpc_model_step(torch.as_tensor(ctx).to("cuda"), torch.as_tensor(tgt).to("cuda"), act, cum=cum,
                          flags=E.EDPC_STEP_UPDATE)
        for s, row, x in zip(act, cum.cpu().numpy().astype(np.int64), tgt):
            coders[s].encode(int(row[x]), int(row[int(x) + 1] - row[x]))
    for s, p in enumerate(pays):
        assert p == (coders[s].finish() if lens[s] else b"")
