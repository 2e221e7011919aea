"""Keys outside the tiles of a row block stay out of its outputs, also where their K and V are not finite (later positions of a
sequence that went wrong there, the unfilled end of a cache): a weight of zero would turn them into NaN in a matrix product."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_04460_amd as vs
import synth
from gpu_util import make_qkv, check_attention, dense_form, lists

pytestmark = pytest.mark.gpu


def _spoilt(k, v, bad):
    k, v = k.clone(), v.clone()
    k[:, bad:] = float("nan")
    v[:, bad:] = float("nan")
    return k, v


def _clean_rows(pos0, n_q, bad, block):
    """Rows of the chunk whose block of `block` rows has no key >= bad in its tiles of 32 keys."""
    r = np.arange(n_q)
    last = np.minimum(pos0 + (r // block + 1) * block, pos0 + n_q) - 1
    return r[last // 32 * 32 + 31 < bad]


def _sample(rows, count=120):
    return rows if len(rows) <= count else np.unique(np.concatenate([rows[:8], rows[-72:], rows[::len(rows) // 40]]))


@pytest.mark.parametrize("hq,hk,n,pos0,n_q,bad", [
    (8, 8, 2048, 0, 2048, 740),                              # 64 rows of a head in a workgroup: behind the workgroup's last tile
    (8, 8, 2048, 0, 2048, 672),                              # the second row block's own tile
    (32, 8, 4096, 2048, 480, 2528),                          # two heads of a group; a chunk with keys behind it
    (18, 9, 2304, 1561, 455, 2016),
    (24, 24, 2048, 0, 2048, 1111),                           # about one round of workgroups
    (8, 2, 6001, 0, 6001, 3456),
    (32, 8, 5000, 3700, 1290, 4992),
])
def test_dense_two_row_blocks_later_keys(hq, hk, n, pos0, n_q, bad):
    """The dense form whose wavefronts own two row blocks and whose stages go past the last tile of either."""
    assert dense_form(hq, hk, n_q, n, pos0) == "duo"
    (q, k, v), (qb, kb, vb) = make_qkv(3000 + bad, hq, hk, n)
    kx, vx = _spoilt(k, v, bad)
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o, lse = torch.empty_like(qc), torch.empty((hq, n_q), dtype=torch.float32, device="cuda")
    vs.dense_prefill(qc, kx, vx, o, lse, pos0=pos0)
    torch.cuda.synchronize()
    clean = _clean_rows(pos0, n_q, bad, 32)
    assert torch.isfinite(o[:, clean].float()).all() and torch.isfinite(lse[:, clean]).all()
    assert o[:, max(bad - pos0, 0):].isnan().all()
    rows = _sample(clean)
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:pos0 + n_q], kb, vb, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


def _sparse_chunk(q, k, v, iv, cv, is_, cs, pos0, n_q, gran=None):
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    hq, hk, n = q.shape[0], k.shape[0], k.shape[1]
    qc = q[:, pos0:pos0 + n_q].contiguous()
    o, lse = torch.empty_like(qc), torch.empty((hq, n_q), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.sparse_prefill_workspace(hq, hk, iv.shape[0], n), dtype=torch.uint8, device="cuda")
    vs.sparse_prefill(qc, k, v, f(iv), f(cv), f(is_), f(cs), o, lse, ws, slash_granularity=gran, pos0=pos0)
    torch.cuda.synchronize()
    return o, lse, ws


@pytest.mark.parametrize("pos0", [1, 31, 37])
def test_sparse_gathered_tile_behind_a_row_block(pos0):
    """A chunk that starts inside a key block: the columns of that key block that lie behind the first row block, but in the chunk, may
    fill a gathered tile of their own.  The first row block neither multiplies nor counts it (a workgroup each)."""
    n, n_q = 256, 64
    cols = list(range(32)) + list(range(pos0 + 32, (pos0 + 31) // 32 * 32 + 32))
    (q, k, v), (qb, kb, vb) = make_qkv(3100 + pos0, 1, 1, n)
    kx, vx = _spoilt(k, v, pos0 + 32)
    iv, cv = lists([cols])
    is_, cs = lists([[n_q + 40]])                            # a far offset only: no key block is listed
    o, lse, ws = _sparse_chunk(q, kx, vx, iv, cv, is_, cs, pos0, n_q)
    rows = np.arange(32)
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:pos0 + n_q], kb, vb, iv, cv, is_, cs, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)
    executed, gathered, staged = vs.sparse_prefill_counters(ws)
    assert (executed, gathered, staged) == (3, 4, 0)


@pytest.mark.parametrize("hq,hk,n", [(1, 1, 1000), (8, 2, 1024),          # a row block to a workgroup
                                     (8, 8, 1055), (8, 2, 3999),          # two, four
                                     (32, 8, 1400), (64, 64, 300)])       # the kernel for many row blocks
@pytest.mark.parametrize("cols", [1, 33, 63, 2433])
def test_sparse_padding_of_gathered_tiles(hq, hk, n, cols):
    """What pads the last gathered tile is not the last key of the sequence, nor any other that the row block does not have."""
    bad = n - 40
    cols = min(cols, bad - 3)
    rng = np.random.default_rng(cols)
    (q, k, v), (qb, kb, vb) = make_qkv(3200 + n, hq, hk, n)
    kx, vx = _spoilt(k, v, bad)
    iv, cv = lists([rng.choice(bad, cols - h % 2 if cols > 1 else cols, replace=False) for h in range(hk)])
    is_, cs = lists([[0, 3, 200]] * hk)
    o, lse, _ = _sparse_chunk(q, kx, vx, iv, cv, is_, cs, 0, n)
    clean = _clean_rows(0, n, bad, 128)
    assert torch.isfinite(o[:, clean].float()).all()
    rows = _sample(clean)
    ref_o, ref_lse = oracle.sparse_attention(qb, kb, vb, iv, cv, is_, cs, rows=rows)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)


@pytest.mark.parametrize("hq,hk,n,pos0,n_q,gran", [
    (1, 1, 1000, 400, 333, None), (8, 2, 4200, 96, 77, 32),              # a row block to a workgroup
    (8, 8, 1300, 100, 1055, None), (32, 8, 4101, 3000, 301, None),       # two
    (8, 2, 4200, 100, 3999, None), (32, 8, 4101, 3009, 700, None),       # four
    (32, 8, 1500, 64, 1411, 32), (32, 8, 1500, 33, 1412, None), (64, 64, 400, 0, 301, None),    # the kernel for many row blocks
    (1, 1, 500, 2, 3, None),
])
def test_keys_behind_a_chunk(hq, hk, n, pos0, n_q, gran):
    """A cache that is longer than what it holds so far: nothing behind the chunk's last position is looked at, by the sparse and by the
    dense call."""
    end = pos0 + n_q
    assert end % 32 != 0 and end < n
    rng = np.random.default_rng(n_q)
    (q, k, v), (qb, kb, vb) = make_qkv(3300 + n_q, hq, hk, n)
    kx, vx = _spoilt(k, v, end)
    near = np.arange(end - 2, min(end + 40, n))              # columns on both sides of the end
    iv, cv = lists([np.unique(np.concatenate([near, rng.choice(n, 60 + h % 2, replace=False)])) for h in range(hk)])
    is_, cs = lists([[0, 1, 3, n // 3]] * hk)
    o, lse, _ = _sparse_chunk(q, kx, vx, iv, cv, is_, cs, pos0, n_q, gran)
    rows = _sample(np.arange(n_q))
    ref_o, ref_lse = oracle.sparse_attention(qb[:, pos0:end], kb, vb, iv, cv, is_, cs, rows=rows, pos0=pos0, granularity=gran or 1)
    assert torch.isfinite(o.float()).all()
    check_attention(o, lse, ref_o, ref_lse, rows=rows)
    qc = q[:, pos0:end].contiguous()
    vs.dense_prefill(qc, kx, vx, o, lse, pos0=pos0)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    ref_o, ref_lse = oracle.dense_attention(qb[:, pos0:end], kb, vb, rows=rows, pos0=pos0)
    check_attention(o, lse, ref_o, ref_lse, rows=rows)
