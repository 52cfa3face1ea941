"""Mutual information on both sides of the line between one kept block of scratch
memory and a block for each matrix: the estimate, the counts and the distances, with
and without the caller's own array of counts, against the same in torch."""

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


@pytest.mark.parametrize("c", [2895, 2896, 4097])
def test_both_sides(E, c):
    v, d = 3, 5
    g = torch.Generator(device="cuda").manual_seed(c)
    z = torch.randn((c, d), device="cuda", generator=g)
    y = z + torch.randn(z.shape, device="cuda", generator=g)
    banner(f"mutual information of {c} samples")
    dz, dy = ((x[:, None] - x[None]).abs().amax(-1) for x in (z, y))  # exact: rounded differences, maxima
    inf = torch.full((c,), float("inf"), device="cuda")
    dz.diagonal().copy_(inf)
    dy.diagonal().copy_(inf)
    eps = torch.maximum(dz, dy).kthvalue(v, 1).values
    counts = torch.stack([(m < eps[:, None]).sum(1) for m in (dz, dy)], 1).int()
    got_c = torch.full((c, 2), -1, dtype=torch.int32, device="cuda")
    got_e = torch.empty(c, device="cuda")
    mi = E.edpc_mutual_info(z, y, v, counts=got_c, eps=got_e)
    assert torch.equal(got_e, eps)
    assert torch.equal(got_c, counts)
    assert E.edpc_mutual_info(z, y, v) == mi
    h = np.concatenate([[0.0], np.cumsum(1.0 / np.arange(1, c + 2))])  # psi(n) = h[n - 1] - gamma
    n = counts.cpu().numpy()
    ref = h[v - 1] + h[c - 1] - (h[n[:, 0]] + h[n[:, 1]]).mean()
    assert abs(mi - ref) <= 1e-12 * c
