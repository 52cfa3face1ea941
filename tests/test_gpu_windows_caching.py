"""Captured windows whose row bucket lies past the size up to which the per-stream
state is cached, with fewer active rows than that: their launches take other kernels of
the FDM than direct steps do.  Both write the same payloads and read each other's."""

import struct
import zlib

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

NO_GRAPHS = 0x20
MODEL = dict(context=16, embed=16, latent=256, blocks=1, hidden=64, branches=2, lr=1e-3, beta1=0.9, beta2=0.999,
             eps=1e-8, seed=4)
# 3 x 4 bytes x 256 x 256 a stream: 213 streams reach 160 MiB, and the bucket of 210 is 256
LENS = [16 + 300] * 210 + [30] * 50


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


def _other(cont):
    """The container with the graphs flag of its configuration turned round."""
    b = bytearray(cont.cpu().numpy().tobytes())
    hl = struct.unpack_from("<I", b, 8)[0]
    struct.pack_into("<I", b, 48, struct.unpack_from("<I", b, 48)[0] ^ NO_GRAPHS)
    struct.pack_into("<I", b, hl - 4, zlib.crc32(bytes(b[:hl - 4])))
    return torch.as_tensor(np.frombuffer(bytes(b), np.uint8).copy()).to("cuda")


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_both_ways(E, precision):
    data = torch.as_tensor(np.random.RandomState(1).randint(97, 105, sum(LENS)).astype(np.uint8)).to("cuda")
    banner(f"windows across the caching line {precision}")
    windows = E.edpc_encode(lib_cfg(E, MODEL, precision), data, LENS)
    direct = E.edpc_encode(lib_cfg(E, MODEL, precision, graphs=False), data, LENS)
    assert torch.equal(_other(direct), windows)
    for c in (_other(windows), _other(direct)):  # coded one way, decoded the other
        assert torch.equal(E.edpc_decode(c)[0], data)
