"""Attention without a row maximum in most stages: scores that leave the maximum of a row block's first stages far behind.  The
rows are then computed again with a maximum in every stage; results are as exact as those of any other row."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_04460_amd as vs
import synth
from gpu_util import bf16_to_f64, check_attention, dense_form, lists, sparse_rows

pytestmark = pytest.mark.gpu

SCALE = 128 ** -0.5


def _inputs(seed, hq, hk, n, growth, big_v=0.0):
    """The score of key n // 2 is `growth` powers of two above those before it, that of key n // 4 half as many, in every second KV head (a
    workgroup without them sits beside one that starts again); big_v: V of key n // 2."""
    q, k, v = synth.qkv(seed, hq, hk, n)
    q, k, v = q.float(), k.float(), v.float()
    q[:, :, 0] = 16.0
    k[:, :, 0] = 0.0
    step = growth / (16.0 * SCALE * 1.4426950408889634)
    k[::2, n // 2, 0] = step
    k[::2, n // 4, 0] = 0.5 * step
    if big_v:
        v[::2, n // 2] = big_v
    q, k, v = (x.bfloat16() for x in (q, k, v))
    return (q.cuda(), k.cuda(), v.cuda()), tuple(synth.to_bits(x) for x in (q, k, v))


def _rows(n):
    """Before, between and after the two keys, first and last rows."""
    return np.unique(np.concatenate([np.arange(4), [n // 4 - 1, n // 4, n // 4 + 1, n // 2 - 1, n // 2, n // 2 + 1], np.arange(n // 2, n, n // 23), [n - 33, n - 2, n - 1]]))


def _check(o, lse, ref_o, ref_lse, rows, big_v):
    if big_v:                                                # rows that hold the large V, relative to it; the others as they are
        large = np.abs(ref_o).max(axis=(0, 2)) > 1e3
        got = bf16_to_f64(o)[:, rows]
        assert np.isfinite(got).all()
        assert np.abs(got[:, large] - ref_o[:, large]).max(initial=0.0) <= 2e-2 * big_v
        assert np.abs(got[:, ~large] - ref_o[:, ~large]).max(initial=0.0) <= 2e-2
    else:
        check_attention(o, lse, ref_o, ref_lse, rows=rows)


# 2^20: kept as it is; 2^50: kept where O is finite; 2^100: sums out of range; 2^300: infinite
GROWTH = [(20, 0.0), (50, 0.0), (50, 2.0 ** 90), (100, 0.0), (300, 0.0)]


@pytest.mark.parametrize("growth,big_v", GROWTH)
@pytest.mark.parametrize("hq,hk,n,form", [(64, 16, 1411, "long"), (160, 160, 600, "long"), (16, 4, 2050, "duo"), (1, 1, 3000, "lone"), (32, 8, 999, "short")])
def test_dense(hq, hk, n, form, growth, big_v):
    assert dense_form(hq, hk, n, n) == form
    (q, k, v), (qb, kb, vb) = _inputs(4000 + n, hq, hk, n, growth, big_v)
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    vs.dense_prefill(q, k, v, o, lse)
    torch.cuda.synchronize()
    rows = _rows(n)
    ref_o, ref_lse = oracle.dense_attention(qb, kb, vb, rows=rows)
    _check(o, lse, ref_o, ref_lse, rows, big_v)


@pytest.mark.parametrize("growth,big_v", GROWTH)
@pytest.mark.parametrize("hq,hk,n,pos0,gran,rows_per_workgroup", [
    (32, 8, 1411, 0, None, 4), (160, 160, 600, 0, None, 4), (32, 8, 1600, 32, 32, 4), (64, 32, 1300, 37, None, 4),
    (8, 2, 3999, 0, None, 4), (20, 20, 1300, 0, None, 2), (32, 8, 4200, 3900, None, 2), (2, 2, 1500, 0, None, 1)])
def test_sparse(hq, hk, n, pos0, gran, rows_per_workgroup, growth, big_v):
    """Columns before, between and after the two keys (more than a stage of them before the first), runs of offsets and scattered ones."""
    n_q = n - pos0
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = _inputs(4100 + n, hq, hk, n, growth, big_v)
    iv, cv = lists([np.union1d([n // 4, n // 2], rng.choice(n, 330, replace=False)) for _ in range(hk)])
    is_, cs = lists([np.union1d(np.arange(70), rng.choice(n, 40, replace=False)) for _ in range(hk)])
    assert sparse_rows(hq, hk, n_q, n, iv.shape[1] + is_.shape[1]) == rows_per_workgroup
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qc = q[:, pos0:].contiguous()
    o, lse = torch.empty_like(qc), torch.empty((hq, n_q), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    tiles = []
    for key in (k, torch.zeros_like(k)):                     # zero scores outgrow nothing; what is executed twice counts once
        vs.sparse_prefill(qc, key, v, f(iv), f(cv), f(is_), f(cs), o if key is k else torch.empty_like(o), lse if key is k else None, ws,
                          slash_granularity=gran, pos0=pos0)
        tiles.append(vs.sparse_prefill_counters(ws))
    assert tiles[0] == tiles[1]
    rows = _rows(n)
    rows = rows[rows >= pos0] - pos0
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:], kb, vb, iv, cv, is_, cs, rows=rows, pos0=pos0, granularity=gran or 1)
    _check(o, lse, ref_o, ref_lse, rows, big_v)
