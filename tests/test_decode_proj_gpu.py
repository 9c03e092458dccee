"""The decode projections at the row counts and shapes where their plan
changes, against the oracle's decode layer by layer over random caches: 1, 8,
9, 16, 17, 32, 33 and 64 rows (the streaming kernel up to 8 rows, the GEMM's
64-row tiles above); K split over workgroups and not; more and fewer weight
rows than the workgroups take at once; weight rows that are not multiples of a
tile; a K that is not a multiple of 64.  Logits and residual within 1e-2 max|ref|
per row (as the other decode tests), two calls bit for bit."""
import numpy as np
import pytest
import torch

from helpers import TOL, ensure_lib, gpu_model, oracle_weights, rel_err, residual_rows, shape_of
from oracle import model as om
from workloads import configs, gen

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def P():
    return ensure_lib()


SHAPES = {
    # odd widths: every last tile is partial, the down projection has K = 1040
    "odd": configs.TINY.replace(n_layers=2, hidden=320, n_q_heads=8, n_kv_heads=2, head_dim=64, ffn=1040, vocab=1003),
    # K split over workgroups in O and down; wide gate|up and lm_head
    "wide": configs.TINY.replace(n_layers=2, hidden=2048, n_q_heads=16, n_kv_heads=2, head_dim=128, ffn=8208,
                                 vocab=16400, qk_norm=True),
}


@pytest.mark.parametrize("name", SHAPES)
@pytest.mark.parametrize("rows", [1, 8, 9, 16, 17, 32, 33, 64])
def test_rows(P, name, rows):
    cfg = SHAPES[name]
    glob, layers = gen.model_weights(cfg, seed=71, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    rng = np.random.default_rng(71)
    pos = [int(v) for v in rng.integers(1, 70, rows)]
    pages = [n // 16 + 1 for n in pos]
    tables = gen.disjoint_block_tables(pages, sum(pages), max(pages), 71, 1)
    pool = gen.kv_pool_normal(cfg.n_layers, sum(pages), 16, cfg.n_kv_heads, cfg.head_dim, 71)
    d_pool, d_bt = pool.to(DEV), torch.tensor(tables, device=DEV)
    ids = gen.token_ids(rows, cfg.vocab, seed=71)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = model.workspace(rows, rows)
    out = [torch.full((rows, cfg.vocab), float("nan"), device=DEV) for _ in range(3)]
    resid = []
    for o in out[:2]:
        model.decode_step(ids.to(DEV), pos, d_bt, d_pool, o, ws, err)
        torch.cuda.synchronize()
        resid.append(residual_rows(ws, rows, cfg.hidden).clone())
    assert int(err.item()) == 0
    assert torch.equal(out[0], out[1]) and torch.equal(resid[0], resid[1])
    if rows <= 8:   # the same step without a workspace
        model.decode_step_static(ids.to(DEV), pos, d_bt, d_pool, out[2], err)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[2])
    g, ls = oracle_weights(glob, layers)
    shp = shape_of(cfg)
    check = range(rows) if rows <= 16 else [0, 15, 16, rows // 2, rows - 2, rows - 1]
    for i in check:
        n = pos[i]
        t = np.arange(n)
        kv = pool[:, :, torch.as_tensor(tables[i][t // 16], dtype=torch.long), torch.as_tensor(t % 16)].double().numpy()
        ref, _, _, r = om.decode(int(ids[i]), n, list(kv[:, 0]), list(kv[:, 1]), g, ls, shp, with_residual=True)
        e = rel_err(out[0][i].double().cpu().numpy(), ref)
        assert e <= TOL, f"row {i} of {rows}: logits rel err {e:.3g}"
        e = rel_err(resid[0][i].double().cpu().numpy(), r)
        assert e <= TOL, f"row {i} of {rows}: residual rel err {e:.3g}"


@pytest.mark.parametrize("counts", [[1, 2, 3, 4, 5, 7, 8], [9, 12, 16, 17, 32, 33, 64]])
def test_rows_do_not_depend_on_their_number(P, counts):
    """A row's logits and residual have the same bits in calls of 1 to 8 rows, and
    in calls of 9 to 64, each in a workspace of just its size.  (O and down
    split K in both; gate|up too in some: their partial sums set what a
    workspace for one row must hold.)"""
    cfg = configs.TINY.replace(n_layers=2, hidden=2048, n_q_heads=16, n_kv_heads=4, head_dim=64, ffn=3072, vocab=512,
                               qk_norm=True)
    glob, layers = gen.model_weights(cfg, seed=72, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    most = max(counts)
    pos = [(5 + 37 * i) % 67 for i in range(most)]
    pages = [n // 16 + 1 for n in pos]
    tables = gen.disjoint_block_tables(pages, sum(pages), max(pages), 72, 1)
    pool = gen.kv_pool_normal(cfg.n_layers, sum(pages), 16, cfg.n_kv_heads, cfg.head_dim, 72, DEV)
    ids = gen.token_ids(most, cfg.vocab, seed=72)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)

    def step(first, n):
        rows = list(range(first, first + n))
        out = torch.full((n, cfg.vocab), float("nan"), device=DEV)
        ws = model.workspace(n, n)
        model.decode_step(ids[rows].to(DEV), [pos[i] for i in rows], torch.tensor(tables[rows], device=DEV), pool.clone(),
                          out, ws, err)
        torch.cuda.synchronize()
        return out, residual_rows(ws, n, cfg.hidden).clone()

    all_out, all_resid = step(0, most)
    for n in counts:
        for first in {0, most - n, (most - n) // 2}:
            out, resid = step(first, n)
            assert torch.equal(resid, all_resid[first:first + n]), f"residuals of rows {first}, +{n}"
            assert torch.equal(out, all_out[first:first + n]), f"logits of rows {first}, +{n}"
    assert int(err.item()) == 0
