"""Attention without a row maximum in most stages: scores that leave the maximum of a row block's first stages far behind.  Such a
stage moves the maximum; results are as exact as those of any other row."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_04460_amd as vs
import synth
from gpu_util import bf16_to_f64, check_attention, dense_form, lists, sparse_rows

pytestmark = pytest.mark.gpu

SCALE = 128 ** -0.5
POWER = 16.0 * SCALE * 1.4426950408889634   # powers of two that a score grows by for 1 in channel 0 of its key


def _inputs(seed, hq, hk, n, growth, big_v=0.0, later=0.0):
    """The score of key n // 2 is `growth` powers of two above those before it, that of key n // 4 half as many, in every second KV head (a
    workgroup without them sits beside one that has them); big_v: V of key n // 2; later: the same of key n - 20, for the last rows."""
    q, k, v = synth.qkv(seed, hq, hk, n)
    q, k, v = q.float(), k.float(), v.float()
    q[:, :, 0] = 16.0
    k[:, :, 0] = 0.0
    k[::2, n // 2, 0] = growth / POWER
    k[::2, n // 4, 0] = 0.5 * growth / POWER
    if later:
        k[::2, n - 20, 0] = later / POWER
    if big_v:
        v[::2, n // 2] = big_v
    q, k, v = (x.bfloat16() for x in (q, k, v))
    return (q.cuda(), k.cuda(), v.cuda()), tuple(synth.to_bits(x) for x in (q, k, v))


def _rows(n):
    """Before, between and after the two keys, first and last rows."""
    return np.unique(np.concatenate([np.arange(4), [n // 4 - 1, n // 4, n // 4 + 1, n // 2 - 1, n // 2, n // 2 + 1], np.arange(n // 2, n, n // 23), [n - 33, n - 20, n - 2, n - 1]]))


def _check(o, lse, ref_o, ref_lse, rows, big_v):
    if big_v:                                                # rows that hold the large V, relative to it; the others as they are
        got, got_lse = bf16_to_f64(o)[:, rows], lse.cpu().numpy().astype(np.float64)[:, rows]
        assert np.isfinite(got).all()
        size = np.abs(ref_o).max(axis=2, keepdims=True)
        assert (np.abs(got - ref_o) <= 2e-2 * np.maximum(size, 1.0)).all()
        assert np.abs(got_lse - ref_lse).max() <= 2e-3
    else:
        check_attention(o, lse, ref_o, ref_lse, rows=rows)


# growth, V of the key, growth of a later key: within the range of one maximum, beyond it, infinite weights; V that overflows O unless the
# maximum moves with the key; the same and then a key that makes all before it small again
GROWTH = [(20, 0.0, 0.0), (27, 2.0 ** 102, 0.0), (50, 0.0, 0.0), (50, 2.0 ** 90, 0.0), (100, 0.0, 0.0), (300, 0.0, 0.0),
          (50, 2.0 ** 90, 85.0), (120, 2.0 ** 10, 125.0), (122, 2.0 ** 10, 240.0)]


@pytest.mark.parametrize("growth,big_v,later", GROWTH)
@pytest.mark.parametrize("hq,hk,n,form", [(64, 16, 1411, "long"), (160, 160, 600, "long"), (16, 4, 2050, "duo"), (1, 1, 3000, "lone"), (32, 8, 999, "short")])
def test_dense(hq, hk, n, form, growth, big_v, later):
    assert dense_form(hq, hk, n, n) == form
    (q, k, v), (qb, kb, vb) = _inputs(4000 + n, hq, hk, n, growth, big_v, later)
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    vs.dense_prefill(q, k, v, o, lse)
    torch.cuda.synchronize()
    rows = _rows(n)
    ref_o, ref_lse = oracle.dense_attention(qb, kb, vb, rows=rows)
    _check(o, lse, ref_o, ref_lse, rows, big_v)


@pytest.mark.parametrize("growth,big_v,later", GROWTH)
@pytest.mark.parametrize("hq,hk,n,pos0,gran,rows_per_workgroup", [
    (32, 8, 1411, 0, None, 4), (160, 160, 600, 0, None, 4), (32, 8, 1600, 32, 32, 4), (64, 32, 1300, 37, None, 4),
    (8, 2, 3999, 0, None, 4), (20, 20, 1300, 0, None, 2), (32, 8, 4200, 3900, None, 2), (2, 2, 1500, 0, None, 1)])
def test_sparse(hq, hk, n, pos0, gran, rows_per_workgroup, growth, big_v, later):
    """Columns before, between and after the two keys (more than a stage of them before the first), runs of offsets and scattered ones."""
    n_q = n - pos0
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = _inputs(4100 + n, hq, hk, n, growth, big_v, later)
    iv, cv = lists([np.union1d([n // 4, n // 2, n - 20], rng.choice(n, 330, replace=False)) for _ in range(hk)])
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


@pytest.mark.parametrize("growth,big_v,later", [g for g in GROWTH if g[2]])
@pytest.mark.parametrize("hq,hk,n,form,late,n_rows", [(64, 16, 1411, "long", 1344, 64), (16, 4, 2050, "duo", 1792, 32)])
def test_dense_search_after_growth(hq, hk, n, form, late, n_rows, growth, big_v, later):
    """The stage on the diagonal looks for a maximum.  Here it starts with the later key, so that every row block of the workgroup has it (and, with two
    row blocks to a wavefront, the wavefront that has key n // 2): none is left whose sum alone shows that a row has grown."""
    assert dense_form(hq, hk, n, n) == form
    (q, k, v), (qb, kb, vb) = _inputs(4200 + n, hq, hk, n, growth, big_v)
    k[::2, late, 0] = later / POWER
    kb = synth.to_bits(k)
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    vs.dense_prefill(q, k, v, o, lse)
    torch.cuda.synchronize()
    rows = np.arange(late, late + n_rows)
    ref_o, ref_lse = oracle.dense_attention(qb, kb, vb, rows=rows)
    _check(o, lse, ref_o, ref_lse, rows, big_v)


@pytest.mark.parametrize("growth,big_v,later", [g for g in GROWTH if g[2]])
@pytest.mark.parametrize("hq,hk", [(32, 8), (160, 160)])
def test_sparse_search_after_growth(hq, hk, growth, big_v, later):
    """The kernel for many row blocks looks for a maximum where only one tile of a stage is live, the third of three gathered ones here; the
    stage before holds the key that has grown."""
    n, late = 1411, 1000
    (q, k, v), (qb, kb, vb) = _inputs(4300, hq, hk, n, growth, big_v)
    k[::2, late, 0] = later / POWER
    kb = synth.to_bits(k)
    rng = np.random.default_rng(hq)
    iv, cv = lists([np.union1d([n // 4, n // 2, late], rng.choice(late, 90, replace=False)) for _ in range(hk)])
    is_, cs = lists([np.arange(100)] * hk)
    assert 64 < cv.min() and cv.max() <= 96 and sparse_rows(hq, hk, n, n, iv.shape[1] + is_.shape[1]) == 4
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(q, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws)
    torch.cuda.synchronize()
    rows = np.arange(late - 3, n, 9)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, rows=rows)
    _check(o, lse, ref_o, ref_lse, rows, big_v)


def _late_keys(seed, hq, hk, n, growth):
    """Keys n // 2 to n // 2 + 2 are alike and `growth` powers of two above all others, whose scores are about -growth."""
    q, k, v = synth.qkv(seed, hq, hk, n)
    q, k = q.float(), k.float()
    q[:, :, 0] = 16.0
    k[:, :, 0] = -growth / POWER
    k[:, n // 2, 0] = 0.0
    k[:, n // 2 + 1:n // 2 + 3] = k[:, n // 2:n // 2 + 1]
    q, k = q.bfloat16(), k.bfloat16()
    return (q.cuda(), k.cuda(), v.cuda()), tuple(synth.to_bits(x) for x in (q, k, v))


def _check_late_keys(o, lse, ref_o, ref_lse, rows):
    """The three keys have a weight of one, as bf16 has it, and lse is a score plus ln 3.  The size of a row is then off by the rounding of its 128 results
    alone, each by at most 2^-9 of itself, so its standard deviation is at most 2^-9 / sqrt(3) * sqrt(sum x^4) / sum x^2, 2^-9 / sqrt(128) for normal values;
    rows of a KV head have all but the same results, so one head may be three times off.  (Weights rounded to bf16 beside a sum that is not: up to 2^-9,
    8e-4 on average.)  lse: half a unit of a sum of products of about 12 (fp32) several
    times over, times the scale: about 1e-7 (an exponent of 40, in fp32: up to 1.3e-6, 7.6e-7 on average)."""
    got = bf16_to_f64(o)[:, rows]
    size = (got * ref_o).sum(2) / (ref_o * ref_o).sum(2)
    assert np.sqrt(np.mean((size - 1.0) ** 2)) <= 3 * 2.0 ** -9 / np.sqrt(128.0)
    err = lse.cpu().numpy().astype(np.float64)[:, rows] - ref_lse
    assert np.sqrt(np.mean(err ** 2)) <= 3e-7


@pytest.mark.parametrize("growth", [14, 41, 55])
@pytest.mark.parametrize("hq,hk,n,form", [(64, 16, 1411, "long"), (16, 4, 2050, "duo"), (1, 1, 3000, "lone"), (32, 8, 999, "short")])
def test_dense_late_maximum_is_exact(hq, hk, n, form, growth):
    assert dense_form(hq, hk, n, n) == form
    (q, k, v), (qb, kb, vb) = _late_keys(4400 + n, hq, hk, n, growth)
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    vs.dense_prefill(q, k, v, o, lse)
    torch.cuda.synchronize()
    rows = np.arange(n // 2 + 200, n, 7)
    _check_late_keys(o, lse, *oracle.dense_attention(qb, kb, vb, rows=rows), rows)


@pytest.mark.parametrize("growth", [14, 41, 55])
@pytest.mark.parametrize("hq,hk,n,rows_per_workgroup", [(32, 8, 1411, 4), (160, 160, 600, 4), (8, 2, 3999, 4), (20, 20, 1300, 2), (2, 2, 1500, 1)])
def test_sparse_late_maximum_is_exact(hq, hk, n, rows_per_workgroup, growth):
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = _late_keys(4500 + n, hq, hk, n, growth)
    iv, cv = lists([np.union1d(np.arange(n // 2, n // 2 + 3), rng.choice(n, 330, replace=False)) for _ in range(hk)])
    is_, cs = lists([np.union1d(np.arange(70), rng.choice(n, 40, replace=False)) for _ in range(hk)])
    assert sparse_rows(hq, hk, n, n, iv.shape[1] + is_.shape[1]) == rows_per_workgroup
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(q, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws)
    torch.cuda.synchronize()
    rows = np.arange(n // 2 + 200, n, 7)
    _check_late_keys(o, lse, *oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, rows=rows), rows)


@pytest.mark.parametrize("growth", [20, 100])
@pytest.mark.parametrize("hq,hk,n", [(32, 8, 1411), (160, 160, 600), (20, 20, 1300)])
def test_sparse_output_in_place_of_q(hq, hk, n, growth):
    """A row block reads its rows of Q before it stores its rows of O, once."""
    rng = np.random.default_rng(n)
    (q, k, v), _ = _inputs(4600 + n, hq, hk, n, growth)
    iv, cv = lists([np.union1d([n // 4, n // 2], rng.choice(n, 330, replace=False)) for _ in range(hk)])
    is_, cs = lists([np.union1d(np.arange(70), rng.choice(n, 40, replace=False)) for _ in range(hk)])
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    o = torch.empty_like(q)
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    for out in (o, q):
        vs.sparse_prefill(q, k, v, f(iv), f(cv), f(is_), f(cs), out, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(o, q)


@pytest.mark.parametrize("n", [129, 160, 192])
def test_dense_row_blocks_that_do_not_exist(n):
    """Three stages, of which a wavefront whose two row blocks lie behind the last position masks none, and keys in the last that are not
    numbers: the wavefronts of a workgroup go through the same stages all the same."""
    hq = 160
    assert dense_form(hq, hq, n, n) == "long"
    (q, k, v), (qb, kb, vb) = _inputs(4700 + n, hq, hq, n, 0.0)
    kx = k.clone()
    kx[:, 128:] = float("nan")
    o, lse = torch.empty_like(q), torch.empty((hq, n), dtype=torch.float32, device="cuda")
    vs.dense_prefill(q, kx, v, o, lse)
    torch.cuda.synchronize()
    rows = np.arange(0, 128, 5)
    check_attention(o, lse, *oracle.dense_attention(qb, kb, vb, rows=rows), rows=rows)
    assert o[:, 128:].isnan().all()
