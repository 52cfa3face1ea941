"""Kraskov kernels at the edges of their tiles and dimension stages: sample
counts around 32 and 64, odd dimensions, rows that are not 16-byte aligned,
equal samples, infinities.  Distances, neighbour distances and counts are
those of the definition evaluated in FP32, bit for bit."""

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


def _reference(z, y, v):
    def dist(x):
        with np.errstate(invalid="ignore"):  # inf - inf is no distance: it counts as 0
            return np.fmax(np.abs(x[:, None] - x[None]), np.float32(0)).max(-1)
    dz, dy = dist(z), dist(y)
    joint = np.maximum(dz, dy)
    off = ~np.eye(len(z), dtype=bool)
    eps = np.array([np.sort(joint[i][off[i]])[v - 1] for i in range(len(z))])
    counts = np.stack([((d < eps[:, None]) & off).sum(1) for d in (dz, dy)], 1)
    return eps, counts


@pytest.mark.parametrize("c,dz,dy,v", [(2, 1, 1, 1), (31, 3, 64, 3), (32, 64, 65, 4), (33, 63, 1, 5),
                                       (65, 130, 16, 16), (100, 20, 36, 7), (513, 5, 68, 2)])
@pytest.mark.parametrize("kind", ["normal", "ties", "infinite"])
def test_edges(E, c, dz, dy, v, kind):
    rng = np.random.default_rng(c + 100 * dz)
    z, y = (rng.standard_normal((c, d)).astype(np.float32) for d in (dz, dy))
    if kind == "ties":
        z, y = np.round(z), np.round(y)
    if kind == "infinite":
        z[::3, 0] = np.inf
        y[1::4, -1] = -np.inf
    eps_r, counts_r = _reference(z, y, v)
    for shift in (0, 1):  # shift 1: the rows start 4 bytes past a 16-byte boundary
        banner(f"mutual information c {c} dims {dz} {dy} v {v} {kind} shift {shift}")
        dev = [torch.zeros(c * x.shape[1] + 4, device="cuda")[shift:shift + x.size].view(c, -1) for x in (z, y)]
        for t, x in zip(dev, (z, y)):
            t.copy_(torch.as_tensor(x))
        counts = torch.empty((c, 2), dtype=torch.int32, device="cuda")
        eps = torch.empty(c, device="cuda")
        E.edpc_mutual_info(dev[0], dev[1], v, counts, eps)
        assert np.array_equal(eps.cpu().numpy(), eps_r)
        assert np.array_equal(counts.cpu().numpy(), counts_r)
