"""Range coder with caller's tables over the number of streams: at the line between
a wave and a thread per stream and past it, payloads equal the integer oracle's
(a sample of the streams) and those of the same streams coded a few at a time."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.rangecoder import RangeEncoder

from .gpu_util import banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("n_steps,n_streams", [(1, 6000), (1, 6001), (5, 6001), (15, 6037), (16, 8000), (16, 8001), (16, 12000),
                                               (16, 12001), (63, 12001), (64, 12001), (64, 24001), (2, 70000)])
def test_streams(E, n_steps, n_streams):
    rng = np.random.default_rng(n_steps + n_streams)
    w = rng.random((61, 256)) ** rng.integers(1, 40, (61, 1))  # flat tables and nearly certain ones
    q = 1 + np.floor(w / w.sum(-1, keepdims=True) * (65536 - 256)).astype(np.int64)
    q[np.arange(61), q.argmax(-1)] += 65536 - q.sum(-1)
    base = np.concatenate([np.zeros((61, 1), np.int64), q.cumsum(-1)], -1)
    pick = rng.integers(0, 61, (n_steps, n_streams))
    sym = np.empty((n_steps, n_streams), np.uint8)
    u = rng.integers(0, 65536, (n_steps, n_streams))
    for k in range(61):
        sym[pick == k] = np.searchsorted(base[k, 1:], u[pick == k], side="right")
    banner(f"coder {n_steps} steps x {n_streams} streams")
    d_cum = torch.as_tensor(base.astype(np.int32)).to("cuda")[torch.as_tensor(pick).to("cuda")]
    d_sym = torch.as_tensor(sym).to("cuda")
    cap = 2 * n_steps + 2
    out, lens = E.edpc_rc_encode(d_cum, d_sym, cap)
    got = out.cpu().numpy()
    for s in {0, 1, 63, 64, n_streams // 2, n_streams - 65, n_streams - 2, n_streams - 1}:
        e = RangeEncoder()
        for t in range(n_steps):
            c, x = base[pick[t, s]], int(sym[t, s])
            e.encode(int(c[x]), int(c[x + 1] - c[x]))
        assert got[s, :lens[s]].tobytes() == e.finish(), s
    few = 1000
    for a in range(0, n_streams, 7 * few):
        o, ln = E.edpc_rc_encode(d_cum[:, a:a + few].contiguous(), d_sym[:, a:a + few].contiguous(), cap)
        assert np.array_equal(ln, lens[a:a + few])
        assert torch.equal(o, out[a:a + few])
    assert torch.equal(E.edpc_rc_decode(d_cum, out, lens), d_sym)
