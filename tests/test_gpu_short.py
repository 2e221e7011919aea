"""GPU parity of the attention kernel for launches with few row blocks (vs_short.hip: the keys of a row block split over four
wavefronts) on both sides of the rules that choose it: sparse calls of up to 128 four-block units with one query head per
workgroup, short chunks of long sequences, dense calls of up to 128 workgroups.  gpu_util states the rules once more, with
the lines read from the sources, so that a case whose kernel changes is noticed.  Bars as everywhere: exact kept-key sets (gpu_util.check_key_set), 2e-2 on bf16 outputs, 2e-3 on the LSE."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_04460_amd as vs
import synth
from gpu_util import (make_qkv, lists, run_sparse, run_dense, check_attention, check_key_set, dense_is_short,
                      sparse_is_short, dense_form, sparse_rows)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gran", [None, 32])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 127, 129, 513])
def test_sparse_tile_edges(n, gran):
    """Fewer tiles than wavefronts, ragged last tiles and stages, row blocks that do not exist."""
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(600 + n, 1, 1, n)
    iv, cv = lists([rng.choice(n, size=max(1, n // 3), replace=False)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=max(1, n // 9), replace=False)]))])
    check_key_set(k, iv, cv, is_, cs, 1, np.arange(n), granularity=gran)
    o, lse, _ = run_sparse(q, k, v, iv, cv, is_, cs, granularity=gran)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, granularity=gran or 1)
    check_attention(o, lse, ref_o, ref_lse)


def test_sparse_several_rounds():
    """One head, n = 16384 (128 units, the last size of the rule): scattered offsets list all 512 key blocks (rounds of 128), and
    5000 columns take several gather rounds (2432 each)."""
    n = 16384
    rng = np.random.default_rng(3)
    (q, k, v), (qb, kb, vb) = make_qkv(61, 1, 1, n)
    iv, cv = lists([rng.choice(n, size=5000, replace=False)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=1500, replace=False)]))])
    rows = synth.sample_rows(3, n, 40, 72, 48)
    check_key_set(k, iv, cv, is_, cs, 1, rows)
    o, lse, _ = run_sparse(q, k, v, iv, cv, is_, cs)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, rows=rows)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


def test_sparse_rows_without_keys():
    """Columns after every row and no offsets: zeros and -inf, from all four partial results."""
    n = 200
    (q, k, v), _ = make_qkv(62, 1, 1, n)
    iv, cv = lists([[150, 199]])
    is_, cs = np.zeros((1, 1), np.int32), np.zeros(1, np.int32)
    o, lse, _ = run_sparse(q, k, v, iv, cv, is_, cs)
    assert (o[0, :150] == 0).all() and torch.isneginf(lse[0, :150]).all() and torch.isfinite(lse[0, 150:]).all()
    assert torch.allclose(o[0, 150:199].float(), v[0, 150].float().expand(49, 128), atol=1e-2)


@pytest.mark.parametrize("hq,hk,n", [(1, 1, 1), (2, 1, 31), (3, 1, 33), (4, 1, 64), (8, 2, 129), (6, 3, 257)])
def test_dense_tile_edges(hq, hk, n):
    (q, k, v), (qb, kb, vb) = make_qkv(700 + n, hq, hk, n)
    o, lse = run_dense(q, k, v)
    ref_o, ref_lse = oracle.dense_attention(qb, kb, vb)
    check_attention(o, lse, ref_o, ref_lse)


@pytest.mark.parametrize("n_q", [1024, 1025])
def test_dense_both_sides_of_the_line(n_q):
    """32 / 8 heads: 1024 rows are 128 workgroups (this kernel), 1025 are 136 (vs_dense.hip)."""
    hq, hk, n = 32, 8, 1100
    (q, k, v), (qb, kb, vb) = make_qkv(63, hq, hk, n)
    pos0 = n - n_q
    qc = q[:, pos0:].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0)
    torch.cuda.synchronize()
    rows = synth.sample_rows(9, n_q, 40, 40, 40)
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:], kb, vb, pos0=pos0)
    check_attention(o, lse, ref_o[:, rows], ref_lse[:, rows], rows=rows)
    assert dense_is_short(hq, hk, n_q, n) == (n_q == 1024)


@pytest.mark.parametrize("hq,hk,n,n_q", [(32, 8, 2051, 256), (8, 2, 700, 33), (4, 2, 513, 1)])
def test_sparse_short_chunk_of_a_group(hq, hk, n, n_q):
    """Several query heads per workgroup: chunks that stay with vs_attention.hip, because the lists are short for 64 units or the
    keys are few."""
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(800 + n, hq, hk, n)
    pos0 = n - n_q
    iv, cv = lists([rng.choice(n, size=n // 10, replace=False) for _ in range(hk)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=60, replace=False)])) for _ in range(hk)])
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qc = q[:, pos0:].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(qc, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws, pos0=pos0)
    torch.cuda.synchronize()
    rows = np.arange(pos0, n)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, rows=rows)
    check_attention(o, lse, ref_o, ref_lse)
    assert not sparse_is_short(hq, hk, n_q, n, iv.shape[1] + is_.shape[1])


@pytest.mark.parametrize("hq,hk,n,n_q,gran", [
    (32, 8, 2400, 256, None),                                # 64 units, the most
    (8, 2, 2100, 33, None),                                  # more than one row block, the second of one row
    (4, 2, 2049, 1, None),                                   # two heads a group, one row
    (6, 3, 2500, 300, None),
    (8, 2, 2176, 64, 32),                                    # tile-granular
    (4, 2, 2143, 31, 32),
])
def test_sparse_short_chunk_edges(hq, hk, n, n_q, gran):
    """Chunks of at most 64 units against at least 2048 keys and 4 times as many as rows, with long lists, take this kernel."""
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(850 + n, hq, hk, n)
    pos0 = n - n_q
    iv, cv = lists([rng.choice(n, size=n // 4, replace=False) for _ in range(hk)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=60, replace=False)])) for _ in range(hk)])
    assert sparse_is_short(hq, hk, n_q, n, iv.shape[1] + is_.shape[1])
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qc = q[:, pos0:].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(qc, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws, slash_granularity=gran, pos0=pos0)
    torch.cuda.synchronize()
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:], kb, vb, iv, cv, is_, cs, granularity=gran or 1, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse)


@pytest.mark.parametrize("hq,hk,n_q,n", [(1, 1, 65, 65), (3, 3, 1, 97), (2, 1, 33, 33), (4, 1, 31, 31), (8, 8, 32, 96), (3, 3, 33, 64), (2, 1, 32, 32)])
def test_dense_few_keys(hq, hk, n_q, n):
    """Both sides of the line of 64 keys for one query head per workgroup and 32 for two."""
    assert dense_is_short(hq, hk, n_q, n) == (n not in (64, 32))
    (q, k, v), (qb, kb, vb) = make_qkv(1400 + n, hq, hk, n)
    pos0 = n - n_q
    qc = q[:, pos0:].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0)
    torch.cuda.synchronize()
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:], kb, vb, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse)


# ---- beyond the lines: the kernels that give a row block to one wavefront ----
@pytest.mark.parametrize("hq,hk,n", [(48, 48, 700), (80, 40, 500), (48, 48, 641), (72, 36, 1025), (64, 16, 513)])
def test_dense_long_form(hq, hk, n):
    """vs_dense.hip with one, two and four query heads per workgroup, ragged last tiles; many heads keep n small."""
    assert not dense_is_short(hq, hk, n, n)
    (q, k, v), (qb, kb, vb) = make_qkv(1000 + n, hq, hk, n)
    o, lse = run_dense(q, k, v)
    ref_o, ref_lse = oracle.dense_attention(qb, kb, vb)
    check_attention(o, lse, ref_o, ref_lse)


@pytest.mark.parametrize("hq,hk,n,pos0,n_q", [(48, 48, 800, 133, 640), (80, 40, 700, 45, 500), (64, 16, 900, 77, 600)])
def test_dense_long_form_chunk(hq, hk, n, pos0, n_q):
    assert not dense_is_short(hq, hk, n_q, n)
    (q, k, v), (qb, kb, vb) = make_qkv(1100 + n, hq, hk, n)
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0)
    torch.cuda.synchronize()
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:pos0 + n_q], kb, vb, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse)


@pytest.mark.parametrize("hq,hk,n,per_q,gran", [
    (48, 48, 333, False, None), (48, 48, 333, False, 32),    # one head a workgroup: tiles of 128 rows, the last of 77
    (40, 40, 511, False, None),                              # more work queues than one layer has
    (48, 12, 300, True, None), (48, 12, 300, True, 32),      # one list per query head
    (160, 80, 150, False, None),                             # 80 work queues: claims look at 64 of them at a time
    (136, 68, 100, False, 32),
])
def test_sparse_long_form(hq, hk, n, per_q, gran):
    """vs_attention.hip: values against the oracle and exact kept-key sets."""
    rng = np.random.default_rng(n + hq)
    (q, k, v), (qb, kb, vb) = make_qkv(1200 + n + hq, hq, hk, n)
    heads = hq if per_q else hk
    iv, cv = lists([rng.choice(n, size=int(rng.integers(1, n // 4)), replace=False) for _ in range(heads)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=int(rng.integers(1, n // 8)), replace=False)]))
                     for _ in range(heads)])
    assert not sparse_is_short(hq, hk, n, n, iv.shape[1] + is_.shape[1], per_q)
    o, lse, _ = run_sparse(q, k, v, iv, cv, is_, cs, granularity=gran)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, granularity=gran or 1)
    check_attention(o, lse, ref_o, ref_lse)
    check_key_set(k, iv, cv, is_, cs, hq, np.arange(n), granularity=gran)


@pytest.mark.parametrize("hq,hk,n,pos0,n_q,per_q,gran", [(48, 48, 500, 77, 300, False, None), (48, 12, 400, 45, 333, True, None),
                                                         (48, 48, 500, 160, 301, False, 32)])
def test_sparse_long_form_chunk(hq, hk, n, pos0, n_q, per_q, gran):
    rng = np.random.default_rng(n + pos0)
    (q, k, v), (qb, kb, vb) = make_qkv(1300 + n, hq, hk, n)
    heads = hq if per_q else hk
    iv, cv = lists([rng.choice(n, size=n // 9, replace=False) for _ in range(heads)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=n // 14, replace=False)])) for _ in range(heads)])
    assert not sparse_is_short(hq, hk, n_q, n, iv.shape[1] + is_.shape[1], per_q)
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, heads, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(qc, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws, slash_granularity=gran, pos0=pos0)
    torch.cuda.synchronize()
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:pos0 + n_q], kb, vb, iv, cv, is_, cs, granularity=gran or 1, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse)


@pytest.mark.parametrize("hq,hk,n,per_q,gran", [
    (8, 8, 1055, False, None),                               # 264 row blocks: two to a workgroup, the last one alone and ragged
    (9, 3, 900, False, 32),                                  # a group of three
    (16, 4, 545, True, None),                                # a mask per query head
])
def test_sparse_two_row_blocks(hq, hk, n, per_q, gran):
    """More than 256 row blocks, at most 128 units: two row blocks share a workgroup; few and many tiles per wavefront."""
    assert 256 < hq * -(-n // 32) <= 512
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(1500 + n, hq, hk, n)
    ih = hq if per_q else hk
    iv, cv = lists([rng.choice(n, size=3 + 40 * (h % 2), replace=False) for h in range(ih)], cap=60)
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=2 + 30 * (h % 3), replace=False)])) for h in range(ih)], cap=70)
    assert sparse_is_short(hq, hk, n, n, 130, per_q) and sparse_rows(hq, hk, n, n, 130, per_q) == 2
    rows = synth.sample_rows(4, n, 40, 40, 60)
    if not per_q:
        check_key_set(k, iv, cv, is_, cs, hq, rows, granularity=gran)
    o, lse, _ = run_sparse(q, k, v, iv, cv, is_, cs, granularity=gran)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, rows=rows, granularity=gran or 1)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n", [(8, 2, 1056), (8, 2, 1024), (9, 9, 929), (6, 6, 1342)])
def test_dense_around_the_line_of_row_blocks(hq, hk, n):
    """256 row blocks (one to a workgroup) and a few more (two: two heads, or 64 rows of one head)."""
    assert dense_is_short(hq, hk, n, n) and abs(hq * -(-n // 32) - 256) <= 14
    assert dense_form(hq, hk, n, n) == ("lone" if hq * -(-n // 32) <= 256 else "short")
    (q, k, v), (qb, kb, vb) = make_qkv(1600 + n, hq, hk, n)
    o, lse = run_dense(q, k, v)
    rows = synth.sample_rows(5, n, 40, 40, 60)
    ref_o, ref_lse = oracle.dense_attention(qb, kb, vb, rows=rows)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n,n_q,gran", [(1, 1, 16384, 333, None), (2, 2, 16416, 96, 32), (4, 1, 9000, 70, None)])
def test_sparse_lone_row_blocks_several_rounds(hq, hk, n, n_q, gran):
    """One row block per workgroup: more than 256 listed key blocks and more than 2432 columns, i.e. several rounds of either list,
    whichever ends first; chunks that start inside a block."""
    assert hq * -(-n_q // 32) <= 256
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(1700 + hq, hq, hk, n)
    pos0 = n - n_q
    iv, cv = lists([rng.choice(n, size=5000 if h == 0 else 40, replace=False) for h in range(hk)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=1500 if hq < 4 else 20, replace=False)])) for _ in range(hk)])
    assert sparse_rows(hq, hk, n_q, n, iv.shape[1] + is_.shape[1]) == 1
    assert sparse_is_short(hq, hk, n_q, n, iv.shape[1] + is_.shape[1])
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qc = q[:, pos0:].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(qc, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws, slash_granularity=gran, pos0=pos0)
    torch.cuda.synchronize()
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:], kb, vb, iv, cv, is_, cs, granularity=gran or 1, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse)


@pytest.mark.parametrize("hq,hk,n_q,n,pos0", [
    (16, 16, 560, 2048, 0),                                  # the first rows: wavefronts without a tile of their own
    (32, 8, 289, 2111, 1822),                                # two heads of a group, odd start, ragged last row block and last tile
    (8, 2, 1030, 2500, 77),
    (9, 9, 929, 4001, 3072),                                 # 64 rows of one head, the second row block missing at the end
    (18, 9, 455, 2048, 1593),
])
def test_dense_two_row_blocks_per_wavefront(hq, hk, n_q, n, pos0):
    """More than 256 row blocks, at most 128 workgroups of the long form, at least 2048 keys."""
    assert hq * -(-n_q // 32) > 256 and dense_is_short(hq, hk, n_q, n) and dense_form(hq, hk, n_q, n, pos0) == "duo"
    (q, k, v), (qb, kb, vb) = make_qkv(1800 + n_q, hq, hk, n)
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0)
    torch.cuda.synchronize()
    rows = synth.sample_rows(7, n_q, 40, 40, 60)
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:pos0 + n_q], kb, vb, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n,pos0,n_q", [(8, 2, 2817, 0, 2817), (32, 8, 2100, 1339, 761), (12, 6, 2049, 0, 2049), (8, 2, 2560, 0, 2560),
                                              (6, 3, 3499, 0, 3499)])
def test_dense_long_keys_many_row_blocks(hq, hk, n, pos0, n_q):
    """At least 2048 keys and about 640 row blocks of grouped heads or more, few keys to a row: a second round of workgroups."""
    assert dense_form(hq, hk, n_q, n, pos0) == "duo"
    (q, k, v), (qb, kb, vb) = make_qkv(1750 + n, hq, hk, n)
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o, lse = torch.full_like(qc, float("nan")), torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0 if n_q != n else None)
    torch.cuda.synchronize()
    rows = synth.sample_rows(8, n_q, 33, 40, 60)
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:pos0 + n_q], kb, vb, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n,pos0,n_q", [(8, 2, 1129, 0, 1129), (8, 2, 2016, 0, 2016), (3, 3, 3201, 0, 3201), (6, 6, 1603, 99, 1500), (1, 1, 8222, 0, 8222)])
def test_dense_lone_row_blocks_second_round(hq, hk, n, pos0, n_q):
    """More than 256 row blocks of one workgroup each: the smallest and the largest number, ragged last row blocks, a chunk."""
    assert 256 < hq * -(-n_q // 32) <= 512 and dense_form(hq, hk, n_q, n, pos0) == "lone"
    (q, k, v), (qb, kb, vb) = make_qkv(1700 + n, hq, hk, n)
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o, lse = torch.full_like(qc, float("nan")), torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0 if n_q != n else None)
    torch.cuda.synchronize()
    rows = synth.sample_rows(6, n_q, 33, 40, 60)
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:pos0 + n_q], kb, vb, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n,pos0,n_q", [(24, 24, 2048, 0, 2048), (8, 2, 6001, 0, 6001), (32, 8, 5000, 3700, 1290),   # evenly spread
                                              (32, 8, 2048, 0, 2048), (32, 8, 2100, 31, 2060)])                            # long form
def test_dense_about_one_round_of_workgroups(hq, hk, n, pos0, n_q):
    """More than 128 workgroups of the long form, at least 2048 keys: spread over two-row-block workgroups where the longest workgroup
    would be all that runs in the end, or not."""
    assert not dense_is_short(hq, hk, n_q, n)
    assert dense_form(hq, hk, n_q, n, pos0) == ("long" if (hq, n) in ((32, 2048), (32, 2100)) else "duo")
    (q, k, v), (qb, kb, vb) = make_qkv(1900 + n, hq, hk, n)
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, k, v, o, lse, pos0=pos0 if n_q != n else None)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    rows = synth.sample_rows(8, n_q, 24, 24, 40)
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:pos0 + n_q], kb, vb, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n,n_q,per_q,gran", [
    (8, 2, 1700, 1700, False, None), (8, 2, 2048, 2048, False, 32),      # two heads of a group share a workgroup
    (32, 8, 4101, 300, False, None),
    (6, 3, 2431, 2431, False, None),                                     # a group of two, 456 row blocks
    (20, 20, 1290, 1290, False, None), (8, 2, 4096, 4096, True, 32),     # one head a workgroup, 220 and 256 units
    (8, 2, 2080, 2080, False, 32), (8, 2, 3999, 3999, False, None),      # four heads of a group, 520 and 1000 row blocks
    (32, 8, 4101, 600, False, None), (12, 6, 1999, 1999, False, None),   # two heads of a group and 64 rows
    (33, 33, 1025, 1025, False, None), (10, 10, 4096, 4096, False, 32),  # 128 rows of one head: 297 and 320 units
    (8, 2, 4128, 4128, False, None), (33, 33, 1190, 1190, False, None),  # just beyond: vs_attention.hip
])
def test_sparse_few_row_blocks(hq, hk, n, n_q, per_q, gran):
    """Up to 1024 row blocks of grouped heads, up to 320 units of one head, at least 1000 rows or 4096 keys: two and four row blocks in
    a workgroup."""
    rng = np.random.default_rng(n + hq)
    (q, k, v), (qb, kb, vb) = make_qkv(2000 + n, hq, hk, n)
    heads, pos0 = hq if per_q else hk, n - n_q
    iv, cv = lists([rng.choice(n, size=5 + 60 * (h % 3), replace=False) for h in range(heads)], cap=130)
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=3 + 40 * (h % 2), replace=False)])) for h in range(heads)], cap=70)
    assert sparse_is_short(hq, hk, n_q, n, 200, per_q) == ((hq, n) not in ((8, 4128), (33, 1190)))
    blocks, units = hq * -(-n_q // 32), hq * -(-n_q // 128)
    alone = per_q or hq == hk
    assert sparse_rows(hq, hk, n_q, n, 200, per_q) == (2 if (units <= 256 if alone else blocks <= 512) else 4)
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qc = q[:, pos0:].contiguous()
    o = torch.full_like(qc, float("nan"))
    lse = torch.full((hq, n_q), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, heads, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(qc, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws, slash_granularity=gran, pos0=pos0 if pos0 else None)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
    rows = synth.sample_rows(6, n_q, 32, 40, 40)
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:], kb, vb, iv, cv, is_, cs, rows=rows, granularity=gran or 1, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)
    if not per_q and not pos0:
        check_key_set(k, iv, cv, is_, cs, hq, rows, granularity=gran)


@pytest.mark.parametrize("hq,hk,n,rows", [
    (8, 2, 1024, 1), (4, 4, 2048, 1), (8, 2, 1056, 2), (9, 9, 929, 2), (8, 8, 4096, 2), (8, 2, 2080, 4), (10, 10, 4096, 4), (33, 33, 1190, 4), (8, 2, 700, 4),
])
def test_sparse_workgroup_that_ran(hq, hk, n, rows):
    """The form that ran, from what it staged: column 0 is one gathered tile per workgroup, whose row blocks are `rows`."""
    (q, k, v), _ = make_qkv(2200 + n, hq, hk, n, rope=False)
    zero, one = torch.zeros((hk, 4), dtype=torch.int32, device="cuda"), torch.ones(hk, dtype=torch.int32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, hk, n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(q, k, v, zero, one, zero, one, torch.empty_like(q), None, ws)
    _, gathered, _ = vs.sparse_prefill_counters(ws)
    assert sparse_rows(hq, hk, n, n, 8) == rows
    group = hq // hk
    hc = min(rows, 4 if group % 4 == 0 else 2 if group % 2 == 0 else 1)
    assert gathered == hq // hc * -(-n // (32 * rows // hc))
