"""Captured step windows: they are only captured where a row bucket lasts, so a
run long enough for that, with a bucket that ends on the way, against the same
steps launched one by one."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

SMALL = dict(context=16, embed=16, latent=64, blocks=2, hidden=128, branches=2, lr=1e-3, beta1=0.9,
             beta2=0.999, eps=1e-8, seed=0)
FLAGS = slice(48, 52)  # configuration flags in the header


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


def _payloads(cont, n):
    b = cont.cpu().numpy().tobytes()
    head = bytearray(b[:92 + 20 * n])
    head[FLAGS] = bytes(4)
    return bytes(head), b[96 + 20 * n:]


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("lens", [[700] * 3, [300] * 130 + [620] * 5, [16 + 255] * 2, [16 + 257] * 2])
def test_windows_equal_direct_steps(E, precision, lens):
    rng = np.random.RandomState(sum(lens))
    data = torch.as_tensor(rng.randint(97, 105, sum(lens)).astype(np.uint8)).to("cuda")
    banner(f"windows {precision} {len(lens)} streams, longest {max(lens)}")
    cont = E.edpc_encode(lib_cfg(E, SMALL, precision), data, lens)
    direct = E.edpc_encode(lib_cfg(E, SMALL, precision, graphs=False), data, lens)
    assert _payloads(cont, len(lens)) == _payloads(direct, len(lens))
    for c in (cont, direct):
        assert torch.equal(E.edpc_decode(c)[0], data)
    # the same steps in calls of odd sizes: windows and direct steps in turn
    s = E.edpc_encoder_begin(lib_cfg(E, SMALL, precision), data, lens)
    for k in (33, 100, 7, 64):
        s.edpc_session_run(k)
    assert torch.equal(s.edpc_encoder_finish(E.edpc_encode_bound(lib_cfg(E, SMALL, precision), lens)), cont)
