"""FP32 products: the tile a product runs on never shows in its results.

A product's sums depend on the MFMA instruction alone, so every tile id of one
instruction (32 x 32, 64 x 32, 32 x 64; and 64 x 64 up to 128 x 128) and every
row count give the same bits for the same row.  A batch is run with each id;
its first rows are run again as a batch of their own.  The row counts are those
where the choice of tile or its edges change, and the first one of each class
is compared with the oracle (bounds 1e-5 and 1e-4: FP32 sums over K <= 256)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.model import Model as OModel

from .gpu_util import banner, lib_cfg, load_oracle_state, oracle_cfg

pytestmark = pytest.mark.gpu

REVISION = 7
# context * embed, hidden and latent that are no multiple of a K chunk or tile
ODD = dict(context=20, embed=16, latent=16, blocks=1, hidden=48, branches=2, lr=1e-3, beta1=0.9,
           beta2=0.999, eps=1e-8, seed=3)
# 2048 outputs: 4096 rows reach the tiles for many rows
WIDE = dict(ODD, context=64, embed=32, hidden=64)


@pytest.fixture(scope="module")
def E():
    import paper_2507_18969_amd as E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return E


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to("cuda")


def _run(E, model, tile, rows, ctx, tgt, **over):
    kid = (REVISION << 48) | sum(tile << (4 * i) for i in range(11))
    m = E.Model(lib_cfg(E, model, "fp32", **over), rows, rows, kid)
    probs = torch.empty((rows, 256), device="cuda")
    m.edpc_model_step(_dev(ctx), _dev(tgt), np.arange(rows), probs=probs,
                      flags=E.EDPC_STEP_BACKWARD | E.EDPC_STEP_KEEP_FDM_GRAD)
    shared = {n: m.edpc_model_read(n, E.EDPC_KIND_GRAD) for n in m.names[:-1]}
    dU = m.edpc_model_read("U", E.EDPC_KIND_GRAD).reshape(rows, -1)
    return probs.cpu().numpy(), shared, dU


def _data(model, rows):
    rng = np.random.RandomState(rows)
    return (rng.randint(97, 123, (rows, model["context"])).astype(np.uint8),
            rng.randint(97, 123, rows).astype(np.uint8))


@pytest.mark.parametrize("branches", [1, 2, 3])
@pytest.mark.parametrize("rows", [1, 17, 200, 1100])
def test_ids_of_one_instruction_give_the_same_bits(E, rows, branches):
    ctx, tgt = _data(ODD, rows)
    for ids in ((0, 1, 2), (3, 4, 5, 6)):
        ref = None
        for tile in ids:
            banner(f"fp32 tile {tile}, {rows} rows, {branches} branches")
            p, g, dU = _run(E, dict(ODD, branches=branches), tile, rows, ctx, tgt)
            if ref is None:
                ref = p, g, dU
                om = OModel(oracle_cfg(dict(ODD, branches=branches)), rows)
                om.round_to_f32()
                c = om.forward(ctx.astype(np.int64), np.arange(rows))
                g_o, dU_o = om.backward(c, tgt.astype(np.int64))
                assert np.abs(p - c["p"]).max() <= 1e-5
                for n, v in g_o.items():
                    assert np.abs(g[n] - v.reshape(-1)).max() <= 1e-4 * np.abs(v).max() + 1e-12, n
                assert np.abs(dU - dU_o.reshape(rows, -1)).max() <= 1e-4 * np.abs(dU_o).max()
            assert np.array_equal(p, ref[0]) and np.array_equal(dU, ref[2])
            for n in g:
                assert np.array_equal(g[n], ref[1][n]), n


@pytest.mark.parametrize("tile", [0, 3])
def test_rows_do_not_depend_on_the_batch(E, tile):
    # 1 / rows scales the adjoint: a power of two, so exactly
    rows, few = 4096, 64
    ctx, tgt = _data(WIDE, rows)
    banner(f"fp32 tile {tile}, {rows} against {few} rows")
    p, _, dU = _run(E, WIDE, tile, rows, ctx, tgt)
    q, _, dV = _run(E, WIDE, tile, few, ctx[:few], tgt[:few])
    assert np.array_equal(p[:few], q)
    assert np.array_equal(dU[:few] * np.float32(rows // few), dV)
