"""Range coder with caller's tables where its kernels have edges: batches of 64
steps, windows of 64 payload bytes, groups of 4 streams, long runs of 0xFF
bytes and carries through them.  Payloads equal the integer oracle's."""

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


def _tables(rng, n_steps, n_streams, flat):
    """Strictly increasing CDFs: nearly flat ones, or with a few large bins."""
    w = rng.random((n_steps, n_streams, 256)) ** (1 if flat else 24)
    q = 1 + np.floor(w / w.sum(-1, keepdims=True) * (65536 - 256)).astype(np.int64)
    big = q.argmax(-1)
    np.put_along_axis(q, big[..., None],
                      np.take_along_axis(q, big[..., None], -1) + 65536 - q.sum(-1, keepdims=True), -1)
    cum = np.zeros((n_steps, n_streams, 257), np.int64)
    cum[..., 1:] = q.cumsum(-1)
    return cum


def _straddle(cum, over):
    """Symbols whose intervals hold the code value 1/2 (so that the bytes pile
    up as 7F FF FF ...), and from step `over` on the last symbol (a carry
    through the pile, if the interval still reaches past 1/2)."""
    low, rng, sym = 0, 1 << 32, []  # the interval [low, low + rng) / 2^(32 + 8 shift)
    half = 1 << 31
    for t, c in enumerate(cum):
        b = [(rng * int(v)) >> 16 for v in c]
        x = 255 if t >= over else max(v for v in range(256) if v == 0 or low + b[v] < half)
        sym.append(x)
        low, rng = low + b[x], b[x + 1] - b[x]
        while rng < (1 << 24):
            low, half, rng = low << 8, half << 8, rng << 8
    return np.array(sym, np.uint8)


@pytest.mark.parametrize("n_steps", [1, 2, 63, 64, 65, 129, 200])
@pytest.mark.parametrize("n_streams", [1, 5, 70])
def test_payloads_equal_the_oracle(E, n_steps, n_streams):
    rng = np.random.default_rng(1000 * n_steps + n_streams)
    cum = _tables(rng, n_steps, n_streams, flat=n_streams == 5)
    u = rng.integers(0, 65536, (n_steps, n_streams))
    sym = (cum[..., 1:] <= u[..., None]).sum(-1).astype(np.uint8)
    for s in range(0, n_streams, 2):
        sym[:, s] = _straddle(cum[:, s], over=n_steps - 1 - s % 7)
    expect = []
    for s in range(n_streams):
        e = RangeEncoder()
        for t in range(n_steps):
            x = int(sym[t, s])
            e.encode(int(cum[t, s, x]), int(cum[t, s, x + 1] - cum[t, s, x]))
        expect.append(e.finish())
    banner(f"coder {n_steps} steps x {n_streams} streams")
    d_cum = torch.as_tensor(cum.astype(np.int32)).to("cuda")
    out, lens = E.edpc_rc_encode(d_cum, torch.as_tensor(sym).to("cuda"), 2 * n_steps + 2)
    got = out.cpu().numpy()
    for s in range(n_streams):
        assert got[s, :lens[s]].tobytes() == expect[s], s
    assert np.array_equal(E.edpc_rc_decode(d_cum, out, lens).cpu().numpy(), sym)
    if n_steps == 200:  # a carry went through a pile of 0xFF: 7F FF FF ... became 80 00 00 ...
        assert expect[0].startswith(b"\x80" + bytes(11))
