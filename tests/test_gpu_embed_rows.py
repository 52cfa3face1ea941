"""Embedding where several rows share a workgroup (below 1024 features, from 2048 rows
on) and where one has it to itself, over rows around those groups.  Without the LTE and without blocks
the head's input is x U, so U = 1 shows the embedded rows, bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from .gpu_util import banner, lib_cfg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


@pytest.mark.parametrize("rows", [1, 17, 2047, 2048, 2049, 2063])
@pytest.mark.parametrize("context,embed", [(4, 16), (8, 16), (4, 32)])
def test_rows_by_the_activation(E, context, embed, rows):
    F = context * embed  # a power of two <= 256: the FDM is F x F
    cfg = dict(context=context, embed=embed, latent=F, blocks=0, hidden=16, branches=1, lr=1e-3, beta1=0.9,
               beta2=0.999, eps=1e-8, seed=5, lte=False)
    banner(f"embedding {context} x {embed}, {rows} rows")
    m = E.Model(lib_cfg(E, cfg), rows, rows)
    m.edpc_model_write("U", np.tile(np.eye(F, dtype=np.float32), (rows, 1, 1)))
    ctx = np.random.RandomState(rows).randint(0, 256, (rows, context)).astype(np.uint8)
    m.edpc_model_step(torch.as_tensor(ctx).to("cuda"), None, np.arange(rows))
    got = m.edpc_model_activation(0, torch.empty(rows * F, device="cuda")).cpu().numpy()
    assert np.array_equal(got.reshape(rows, F), m.edpc_model_read("emb").reshape(256, embed)[ctx].reshape(rows, F))


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("context,embed", [(12, 16), (20, 16), (36, 16), (60, 16), (64, 16), (68, 16), (20, 64)])
def test_rows_among_others(E, context, embed, precision):
    """Widths that do not divide 1024: a row's probabilities do not depend on the
    rows beside it or on how many there are."""
    cfg = dict(context=context, embed=embed, latent=16, blocks=0, hidden=16, branches=1, lr=1e-3, beta1=0.9,
               beta2=0.999, eps=1e-8, seed=5)
    rows = 2050
    banner(f"embedding {context} x {embed} {precision}")
    m = E.Model(lib_cfg(E, cfg, precision), rows, rows)
    ctx = torch.as_tensor(np.random.RandomState(3).randint(0, 256, (rows, context)).astype(np.uint8)).to("cuda")
    probs = torch.empty(rows, 256, device="cuda")
    m.edpc_model_step(ctx, None, np.arange(rows), probs=probs)
    for a in list(range(0, 60, 7)) + [2030]:
        few = torch.empty(7, 256, device="cuda")
        m.edpc_model_step(ctx[a:a + 7].clone(), None, np.arange(a, a + 7), probs=few)
        assert torch.equal(few, probs[a:a + 7]), a


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("context,embed", [(64, 16), (68, 16), (132, 16), (64, 64), (256, 64)])
def test_wide_rows(E, context, embed, precision):
    """Wide rows: shared out over workgroups up to 512 rows, whole past that."""
    cfg = dict(context=context, embed=embed, latent=16, blocks=0, hidden=16, branches=1, lr=1e-3, beta1=0.9,
               beta2=0.999, eps=1e-8, seed=5)
    rows = 513
    banner(f"embedding {context} x {embed} {precision}, wide rows")
    m = E.Model(lib_cfg(E, cfg, precision), rows, rows)
    ctx = torch.as_tensor(np.random.RandomState(4).randint(0, 256, (rows, context)).astype(np.uint8)).to("cuda")
    whole = torch.empty(rows, 256, device="cuda")
    m.edpc_model_step(ctx, None, np.arange(rows), probs=whole)
    for a, n in ((0, 1), (500, 13), (0, 512)):
        part = torch.empty(n, 256, device="cuda")
        m.edpc_model_step(ctx[a:a + n].clone(), None, np.arange(a, a + n), probs=part)
        assert torch.equal(part, whole[a:a + n]), (a, n)
