"""Wave reductions by lane swaps and DPP, through the head: logits whose largest,
whose sum and whose running sums come from chosen lanes (each distance of the
butterfly), as a range of biases on a model without other signal.  The CDF is
whole numbers, so it has to be the oracle's formula exactly where the
probabilities are; probabilities to FP32 rounding (1e-6)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")


from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu

CFG = dict(context=4, embed=16, latent=16, blocks=0, hidden=16, branches=2, lr=1e-3, beta1=0.9,
           beta2=0.999, eps=1e-8, seed=1, zero_head=True)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("peak", [0, 1, 2, 4, 7, 8, 31, 63, 64, 127, 128, 200, 255])
def test_head_of_a_bias(E, peak):
    banner(f"head, largest logit at {peak}")
    m = E.Model(lib_cfg(E, CFG), 3, 3)
    z = np.random.RandomState(peak).standard_normal(256).astype(np.float32)
    z[peak] = 6.0
    m.edpc_model_write("wh", np.zeros(256 * 64, np.float32))
    m.edpc_model_write("bh", z)
    ctx = torch.zeros(3, 4, dtype=torch.uint8, device="cuda")
    p = torch.empty(3, 256, device="cuda")
    cum = torch.empty(3, 257, dtype=torch.int32, device="cuda")
    m.edpc_model_step(ctx, None, np.arange(3), probs=p, cum=cum)
    z64 = z.astype(np.float64)
    want = np.exp(z64 - z64.max())
    want /= want.sum()
    for r in range(3):
        got = p[r].cpu().numpy()
        assert np.abs(got - want).max() <= 1e-6
        c = cum[r].cpu().numpy().astype(np.int64)
        q = 1 + np.floor(got * np.float32(65280)).astype(np.int64)
        q[np.argmax(q)] += 65536 - q.sum()
        assert np.array_equal(np.diff(c), q) and c[0] == 0 and c[256] == 65536
