"""Prefill at the row counts where the GEMMs change their tile or K split,
against the oracle end to end: the limits of the 64-, 128-, 192- and 256-row
tiles of launches of at most 256 rows (gate|up with 128- and with 256-wide
tiles, O and down with and without a K split; few columns without a split, which
take narrower tiles or two M tiles from 65 rows on), and a few hundred rows, which
take 128-row tiles above 256.  K/V of both layers within 1e-2 max|ref| (the
bf16 bound of the other prefill tests).  Lengths on one side of 256 rows agree bit for bit: above it in
everything, up to it in layer 0, which the projection alone decides (attention
over so few rows splits its keys by the row count)."""
import numpy as np
import pytest
import torch

from helpers import TOL, empty_pool, ensure_lib, gpu_model, kv_logical, oracle_weights, rel_err, shape_of
from oracle import model as om
from workloads import configs, gen

pytestmark = pytest.mark.gpu
DEV = "cuda"
ROWS = [1, 64, 65, 128, 129, 192, 193, 256, 257, 320, 500]
SHAPES = {
    "wide": configs.TINY.replace(hidden=256, n_q_heads=4, n_kv_heads=2, ffn=16448, vocab=512),
    "deep": configs.TINY.replace(hidden=1024, n_q_heads=32, n_kv_heads=4, ffn=4112, vocab=512, qk_norm=True),
    # 5120 Q|K|V columns: 128 x 96 tiles at 500 rows, the last row and column tile partial
    "broad": configs.TINY.replace(hidden=320, n_q_heads=64, n_kv_heads=8, head_dim=64, ffn=1040, vocab=512),
}


@pytest.fixture(scope="module")
def P():
    return ensure_lib()


@pytest.mark.parametrize("name", SHAPES)
def test_row_counts(P, name):
    cfg = SHAPES[name]
    glob, layers = gen.model_weights(cfg, seed=81, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    ids = gen.token_ids(max(ROWS), cfg.vocab, seed=81)
    g, ls = oracle_weights(glob, layers)
    K, V, _ = om.prefill(ids.tolist(), g, ls, shape_of(cfg))      # causal: the rows of every length
    bt = gen.block_table(32, 40, 32, 81, 1)
    d_bt = torch.tensor(bt[None], device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    got = {}
    for n in ROWS:
        pool = empty_pool(cfg, 40, fill_bits=0)
        model.prefill_prefix(ids[:n].to(DEV), [0, n], d_bt, pool, model.workspace(n), err)
        torch.cuda.synchronize()
        got[n] = kv_logical(pool, bt, n)
        for l in range(cfg.n_layers):
            for kv, ref in ((0, K[l][:n]), (1, V[l][:n])):
                e = rel_err(got[n][l, kv], ref)
                assert e <= TOL, f"{n} rows, layer {l} {'KV'[kv]}: {e:.3g}"
    assert int(err.item()) == 0
    few = [n for n in ROWS if n <= 256]
    for n in few:
        np.testing.assert_array_equal(got[n][0], got[256][0, :, :n])
    for n in [n for n in ROWS if n > 256]:
        np.testing.assert_array_equal(got[n], got[500][:, :, :n])
