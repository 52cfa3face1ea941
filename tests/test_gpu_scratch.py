"""Scratch memory kept between synchronous calls: calls of changing sizes, from
several threads and streams, give what each gives alone."""

import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


def test_threads_and_streams(E):
    sizes = [40, 3000, 65, 1024, 130, 2500, 33, 700]  # up to 72 MB: past what is kept
    xs = []
    for c in sizes:
        g = torch.Generator(device="cuda").manual_seed(c)
        z = torch.randn((c, 24), device="cuda", generator=g)
        xs.append((z, z + torch.randn(z.shape, device="cuda", generator=g)))
    banner("mutual information, one thread")
    alone = [E.edpc_mutual_info(z, y) for z, y in xs]
    got = {}

    def work(t):
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        for r in range(3):
            for i in np.random.RandomState(10 * t + r).permutation(len(xs)):
                got[t, r, i] = E.edpc_mutual_info(*xs[i], stream=s)

    banner("mutual information, four threads")
    torch.cuda.synchronize()
    th = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert len(got) == 4 * 3 * len(xs)
    for (t, r, i), v in got.items():
        assert v == alone[i]
