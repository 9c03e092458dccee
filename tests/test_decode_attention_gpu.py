"""Decode attention at the sizes where its work split changes, against the
oracle's decode over the same random caches: 32-key blocks, 128-key splits and
their multiples, one split (no merge) and sixteen, workgroups of four waves and
of two (where more than 256 are needed), runs of one split and of several,
head_dim 64 and 128, groups of 1, 2, 4 and 8 query heads.  Unwritten slots hold NaN patterns; table entries
outside the pool mask their keys.  Residual and logits within
max|gpu - ref| <= 1e-2 max|ref| per row (the bf16 bound of the other decode
tests); the K/V written within it too, and nothing else in the pool changed.
Then what several rows of a call may share, and what a row's bits depend on."""
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


CASES = [
    # head_dim, group, KV heads, positions
    (128, 8, 2, [0, 1, 31, 32, 33, 127, 128, 129]),
    (128, 4, 2, [255, 256, 257, 2047, 2048, 2049]),
    (128, 1, 4, [63, 300, 900, 4000]),
    (64, 2, 2, [0, 31, 64, 127, 128, 1100]),
    (64, 8, 1, [500, 2048, 5000]),
    (128, 8, 8, [1000 + 97 * i for i in range(10)]),     # more than 256 workgroups
    (64, 4, 8, [700 + 131 * i for i in range(12)]),
]


@pytest.mark.parametrize("d,group,hkv,pos", CASES)
def test_split_edges(P, d, group, hkv, pos):
    cfg = configs.TINY.replace(n_layers=1, hidden=256, n_q_heads=group * hkv, n_kv_heads=hkv, head_dim=d, ffn=256,
                               vocab=512, qk_norm=True, name="edges")
    glob, layers = gen.model_weights(cfg, seed=61, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    pages = [n // 16 + 1 for n in pos]
    tables = gen.disjoint_block_tables(pages, sum(pages) + 3, max(pages), 61, 1)
    pool = gen.kv_pool_normal(1, sum(pages) + 3, 16, hkv, d, 61)
    bad = {}                              # sequence -> a page of it that is not in the pool
    for i, n in enumerate(pos):
        slots = torch.arange(n % 16, 16)  # unwritten: quiet NaNs
        pool.view(torch.int16)[:, :, tables[i, n // 16], slots] = gen.SENTINEL_BITS
        if n > 400 and i % 2:
            bad[i] = (n // 16) // 2
            tables[i, bad[i]] = -1 if i % 4 == 1 else sum(pages) + 3
    d_pool = pool.to(DEV)
    ids = gen.token_ids(len(pos), cfg.vocab, seed=61).numpy()
    logits = torch.empty((len(pos), cfg.vocab), dtype=torch.float32, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = model.workspace(len(pos), len(pos))
    for _ in range(2):                    # the second step finds what the first left
        model.decode_step(torch.tensor(ids, dtype=torch.int32, device=DEV), pos,
                          torch.tensor(tables, device=DEV), d_pool, logits, ws, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0           # only the store of slot n reports its page
    resid = residual_rows(ws, len(pos), cfg.hidden).double().cpu().numpy()
    got_pool = d_pool.cpu()
    g, ls = oracle_weights(glob, layers)
    shp = shape_of(cfg)
    for i, n in enumerate(pos):
        keep = [t for t in range(n) if t // 16 != bad.get(i)]
        pg = tables[i][np.array(keep, dtype=int) // 16] if keep else np.zeros(0, dtype=int)
        sl = np.array(keep, dtype=int) % 16
        kv = pool[0][:, torch.as_tensor(pg, dtype=torch.long), torch.as_tensor(sl)].double().numpy()
        ref, k_new, v_new, r = om.decode(int(ids[i]), n, [kv[0]], [kv[1]], g, ls, shp, with_residual=True)
        e = rel_err(logits[i].double().cpu().numpy(), ref)
        assert e <= TOL, f"position {n}: logits rel err {e:.3g}"
        e = rel_err(resid[i], r)
        assert e <= TOL, f"position {n}: residual rel err {e:.3g}"
        at = got_pool[0][:, tables[i, n // 16], n % 16].double().numpy()
        assert rel_err(at[0], k_new[0]) <= TOL and rel_err(at[1], v_new[0]) <= TOL
        got_pool[0][:, tables[i, n // 16], n % 16] = pool[0][:, tables[i, n // 16], n % 16]
    assert torch.equal(got_pool.view(torch.int16), pool.view(torch.int16)), "slots written besides the rows' own"


def test_slot_outside_the_pool(P):
    """The page of slot n is not in the pool: nothing is stored, the token does
    not see its own K/V, and the error word says so."""
    cfg = configs.TINY.replace(n_layers=1, vocab=512, name="edges")
    glob, layers = gen.model_weights(cfg, seed=62, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    n = 160
    tables = gen.disjoint_block_tables([11], 16, 11, 62, 1)
    tables[0, 10] = 16
    pool = gen.kv_pool_normal(1, 16, 16, cfg.n_kv_heads, cfg.head_dim, 62)
    d_pool = pool.to(DEV)
    logits = torch.empty((1, cfg.vocab), dtype=torch.float32, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = model.workspace(1, 1)
    model.decode_step(torch.tensor([5], dtype=torch.int32, device=DEV), [n], torch.tensor(tables, device=DEV),
                      d_pool, logits, ws, err)
    torch.cuda.synchronize()
    assert int(err.item()) == 1
    assert torch.equal(d_pool.cpu().view(torch.int16), pool.view(torch.int16))
    assert torch.isfinite(logits).all()


# Rows of one call that read slots which other rows of it write: (head_dim,
# group, KV heads, tables, positions); rows with one table are one sequence.
SHARED = {
    # three tokens of one sequence, the last two on a new page
    "three": (128, 8, 2, [0, 0, 0], [303, 304, 305]),
    # within one page and one block, from position zero on, in any order
    "start": (64, 2, 2, [0, 0, 0, 0], [2, 0, 3, 1]),
    # two sequences of two and five tokens, over a split's edge, and one row by itself
    "two": (128, 4, 8, [0, 1, 0, 1, 1, 2, 1, 1], [1022, 127, 1023, 128, 129, 40, 130, 131]),
    # 64 tokens: every slot of some blocks comes from the call
    "many": (64, 8, 8, [0] * 64, list(range(1000, 1064))),
    "few keys": (128, 1, 4, [0] * 33, list(range(33))),
}


@pytest.mark.parametrize("name", SHARED)
def test_rows_of_one_sequence(P, name):
    """Several tokens of a sequence in one call: a row attends to the K/V of
    the rows before it, whichever workgroup stores them, as when each token
    has a call of its own (the oracle's decode, token by token)."""
    d, group, hkv, of, pos = SHARED[name]
    cfg = configs.TINY.replace(n_layers=2, hidden=256, n_q_heads=group * hkv, n_kv_heads=hkv, head_dim=d, ffn=256,
                               vocab=512, qk_norm=True, name="shared")
    glob, layers = gen.model_weights(cfg, seed=63, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    ends = [max(n for n, o in zip(pos, of) if o == q) + 1 for q in range(max(of) + 1)]
    pages = [(e + 15) // 16 for e in ends]
    tables = gen.disjoint_block_tables(pages, sum(pages) + 3, max(pages), 63, 1)
    pool = gen.kv_pool_normal(2, sum(pages) + 3, 16, hkv, d, 63)
    for n, o in zip(pos, of):             # what the call writes holds NaN patterns before
        pool.view(torch.int16)[:, :, tables[o, n // 16], n % 16] = gen.SENTINEL_BITS
    d_pool = pool.to(DEV)
    ids = gen.token_ids(len(pos), cfg.vocab, seed=63).numpy()
    logits = torch.empty((len(pos), cfg.vocab), dtype=torch.float32, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    model.decode_step(torch.tensor(ids, dtype=torch.int32, device=DEV), pos, torch.tensor(tables[of], device=DEV),
                      d_pool, logits, model.workspace(len(pos), len(pos)), err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    got_pool, got = d_pool.cpu(), logits.double().cpu().numpy()
    g, ls = oracle_weights(glob, layers)
    shp = shape_of(cfg)
    caches = []
    for q, e in enumerate(ends):
        t = np.arange(e)
        kv = pool[:, :, torch.as_tensor(tables[q][t // 16], dtype=torch.long), torch.as_tensor(t % 16)].double().numpy()
        caches.append(kv)
    for i in sorted(range(len(pos)), key=lambda i: pos[i]):
        n, kv = pos[i], caches[of[i]]
        ref, k_new, v_new = om.decode(int(ids[i]), n, list(kv[:, 0]), list(kv[:, 1]), g, ls, shp)
        e = rel_err(got[i], ref)
        assert e <= TOL, f"row {i}, position {n}: logits rel err {e:.3g}"
        for l in range(2):
            kv[l, 0, n], kv[l, 1, n] = k_new[l][0], v_new[l][0]
            at = got_pool[l][:, tables[of[i], n // 16], n % 16].double().numpy()
            assert rel_err(at[0], k_new[l][0]) <= TOL and rel_err(at[1], v_new[l][0]) <= TOL
    if len(pos) <= 8:                     # the same bits as a call per token
        d_pool = pool.to(DEV)
        for i in sorted(range(len(pos)), key=lambda i: pos[i]):
            model.decode_step(torch.tensor(ids[i:i + 1], dtype=torch.int32, device=DEV), [pos[i]],
                              torch.tensor(tables[of[i]][None], device=DEV), d_pool, logits[:1], model.workspace(1, 1), err)
            torch.cuda.synchronize()
            assert np.array_equal(logits[0].double().cpu().numpy(), got[i]), f"row {i}, position {pos[i]}"
        assert torch.equal(d_pool.cpu().view(torch.int16), got_pool.view(torch.int16))


# head_dim, group, KV heads, positions.  Alone a row runs in workgroups of four
# waves and one split each.  Beside others: two waves with one split, and with
# one, two and four; the same at head_dim 64; four waves with two and with four.
BATCHES = [
    (128, 2, 16, [300, 1000, 2500, 6000, 9000, 40, 127, 0]),
    (64, 4, 4, [4095, 4096, 16383, 2047, 129, 8200, 700, 15000]),
    (128, 1, 8, [1000, 1500, 2047, 1800, 120, 900, 511, 2000]),
    (64, 8, 8, [1000, 1500, 2047, 1800, 120, 900, 511, 2000]),
]


@pytest.mark.parametrize("d,group,hkv,pos", BATCHES)
def test_a_row_does_not_depend_on_its_batch(P, d, group, hkv, pos):
    """A row of up to 8 has the same bits alone, beside others and in another
    order: its splits follow from its own position, and every division of them
    over workgroups and waves merges the same partials in the same tree."""
    cfg = configs.TINY.replace(n_layers=2, hidden=256, n_q_heads=group * hkv, n_kv_heads=hkv, head_dim=d, ffn=256,
                               vocab=512, qk_norm=True, name="batch")
    glob, layers = gen.model_weights(cfg, seed=64, gain_sigma=0.1)
    model = gpu_model(P, cfg, glob, layers)
    pages = [n // 16 + 1 for n in pos]
    tables = gen.disjoint_block_tables(pages, sum(pages), max(pages), 64, 1)
    pool = gen.kv_pool_normal(2, sum(pages), 16, hkv, d, 64, DEV)
    ids = gen.token_ids(len(pos), cfg.vocab, seed=64)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)

    def step(rows):
        out = torch.full((len(rows), cfg.vocab), float("nan"), device=DEV)
        mine = pool.clone()
        ws = model.workspace(len(rows), len(rows))
        model.decode_step(ids[rows].to(DEV), [pos[i] for i in rows], torch.tensor(tables[rows], device=DEV), mine, out,
                          ws, err)
        torch.cuda.synchronize()
        resid = residual_rows(ws, len(rows), cfg.hidden)
        new = [mine[:, :, tables[i, pos[i] // 16], pos[i] % 16].clone() for i in rows]
        return {i: (out[k], resid[k].clone(), new[k]) for k, i in enumerate(rows)}

    alone = {i: step([i])[i] for i in range(len(pos))}
    for rows in ([0, 1], [4, 2], [6, 3, 0, 7, 1], list(range(8)), list(reversed(range(8)))):
        got = step(rows)
        for i in rows:
            for what, a, b in zip(("logits", "residual", "K/V"), got[i], alone[i]):
                assert torch.equal(a, b), f"{what} of position {pos[i]} beside {[pos[k] for k in rows]}"
    assert int(err.item()) == 0
