"""GPU parity of vs_aggregate (vertical-slash aggregation of the dense attention map and Attention Recall) against the
fp64 oracle, through the C ABI.  Tolerance: the aggregated vectors are probability distributions like the indexer's
scores, so they get the same bar (1e-3 relative, plus 1e-7 absolute for entries that are almost zero); the recall, a
single mass in [0, 1], gets 1e-4 absolute."""
import numpy as np
import pytest
import torch

import paper_2603_04460_amd as vs
import synth
from oracle import vs_oracle as oracle
from gpu_util import make_qkv, lists, run_dense

pytestmark = pytest.mark.gpu

REL, ABS, RECALL_ABS = 1e-3, 1e-7, 1e-4


def _dev_lists(iv, cv, is_, cs):
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    return f(iv), f(cv), f(is_), f(cs)


def _run(q, k, out_heads, lse=None, mask=None):
    hq, n, _ = q.shape
    hk = k.shape[0]
    index_heads = 0 if mask is None else mask[0].shape[0]
    ws = torch.empty(vs.aggregate_workspace(hq, hk, index_heads, n), dtype=torch.uint8, device="cuda")
    a_v = torch.full((out_heads, n), float("nan"), dtype=torch.float32, device="cuda")
    a_s = torch.full((out_heads, n), float("nan"), dtype=torch.float32, device="cuda")
    rec = None
    dl = None
    if mask is not None:
        rec = torch.full((out_heads,), float("nan"), dtype=torch.float32, device="cuda")
        dl = _dev_lists(*mask)
    vs.aggregate(q, k, a_v, a_s, ws, lse=lse, lists=dl, recall=rec)
    torch.cuda.synchronize()
    return (a_v.cpu().numpy().astype(np.float64), a_s.cpu().numpy().astype(np.float64),
            None if rec is None else rec.cpu().numpy().astype(np.float64))


def _oracle(qb, kb, group, mask=None):
    hq = qb.shape[0]
    av, as_, rec = [], [], []
    for h in range(hq):
        g = h // group
        if mask is None:
            a, b = oracle.vs_aggregate(qb[h], kb[g])
        else:
            iv, cv, is_, cs = mask
            ih = h if iv.shape[0] == hq else g
            a, b, r = oracle.vs_aggregate(qb[h], kb[g], idx_v=iv[ih, :cv[ih]], idx_s=is_[ih, :cs[ih]])
            rec.append(r)
        av.append(a); as_.append(b)
    return np.stack(av), np.stack(as_), np.array(rec)


def _close(got, ref):
    assert np.isfinite(got).all()
    err = np.abs(got - ref)
    bad = err > REL * np.abs(ref) + ABS
    assert not bad.any(), "worst: got %.6g ref %.6g" % (got[bad][0], ref[bad][0])


@pytest.mark.parametrize("hq,hk,n", [(1, 1, 1), (1, 1, 33), (4, 1, 64), (2, 1, 257), (8, 2, 700), (4, 4, 1000), (4, 1, 2100)])
def test_aggregate_per_query_head(hq, hk, n):
    """Ragged lengths on both sides of the 256-key workgroup and the 64-row stage; each vector sums to 1."""
    (q, k, v), (qb, kb, vb) = make_qkv(300 + n, hq, hk, n)
    a_v, a_s, _ = _run(q, k, hq)
    ref_v, ref_s, _ = _oracle(qb, kb, hq // hk)
    _close(a_v, ref_v)
    _close(a_s, ref_s)
    assert np.abs(a_v.sum(axis=1) - 1).max() < 1e-4 and np.abs(a_s.sum(axis=1) - 1).max() < 1e-4


@pytest.mark.parametrize("n", [31, 32, 65, 191, 225, 289, 545, 1569])
def test_aggregate_tile_edges(n):
    """Lengths around the 32-row tile, a wavefront's two blocks, the 256-row workgroup and the 512-entry diagonal rings, with
    the recall of a mask whose offsets start and end inside a tile."""
    hq, hk = 2, 1
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(500 + n, hq, hk, n, local=True)
    iv, cv = lists([np.sort(rng.choice(n, max(1, n // 20), replace=False))])
    is_, cs = lists([np.unique(np.clip(np.concatenate([[0, 1, 31, 32, 33], np.arange(n // 2, n // 2 + 20), [n - 1]]), 0, n - 1))])
    a_v, a_s, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    ref_v, ref_s, ref_r = _oracle(qb, kb, hq // hk, mask=(iv, cv, is_, cs))
    _close(a_v, ref_v)
    _close(a_s, ref_s)
    assert np.abs(rec - ref_r).max() <= RECALL_ABS, (rec, ref_r)


@pytest.mark.parametrize("hq,hk,n", [(32, 8, 1057), (16, 4, 2085)])
def test_aggregate_many_groups(hq, hk, n):
    """144 groups of 256 resident rows, several workgroups to a group."""
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(520 + n, hq, hk, n, local=True)
    iv, cv = lists([rng.choice(n, 40, replace=False) for _ in range(hk)])
    is_, cs = lists([np.unique(np.concatenate([np.arange(20), rng.choice(n, 30, replace=False)])) for _ in range(hk)])
    a_v, a_s, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    ref_v, ref_s, ref_r = _oracle(qb, kb, hq // hk, mask=(iv, cv, is_, cs))
    _close(a_v, ref_v)
    _close(a_s, ref_s)
    assert np.abs(rec - ref_r).max() <= RECALL_ABS, (rec, ref_r)


@pytest.mark.parametrize("pairs,n", [(103, 1100), (129, 900), (52, 1500), (26, 1500), (85, 1025)])
def test_aggregate_group_sharing(pairs, n):
    """One workgroup per group of 256 resident rows (more than 1024 groups: 206 x 5, 258 x 4) and two (624; 850, with a last group
    of one row; 312), with a recall, per query head and as the mean over a KV group: two query heads of one KV head, repeated."""
    groups = 2 * pairs * -(-n // 256)
    assert (groups > 1024) == (pairs in (103, 129)) and (512 < groups <= 1024) == (pairs in (52, 85))
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(560 + n, 2, 1, n, local=True)
    iv, cv = lists([rng.choice(n, size=n // 10, replace=False)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=n // 20, replace=False)]))])
    ref_v, ref_s, ref_r = _oracle(qb, kb, 2, mask=(iv, cv, is_, cs))
    qr, kr = q.repeat(pairs, 1, 1).contiguous(), k.repeat(pairs, 1, 1).contiguous()
    mask = (np.repeat(iv, pairs, 0), np.repeat(cv, pairs), np.repeat(is_, pairs, 0), np.repeat(cs, pairs))
    a_v, a_s, rec = _run(qr, kr, 2 * pairs, mask=mask)
    _close(a_v, np.tile(ref_v, (pairs, 1)))
    _close(a_s, np.tile(ref_s, (pairs, 1)))
    assert np.abs(rec - np.tile(ref_r, pairs)).max() <= RECALL_ABS
    a_v, a_s, _ = _run(qr, kr, pairs)
    _close(a_v, np.repeat(ref_v.mean(0, keepdims=True), pairs, 0))
    _close(a_s, np.repeat(ref_s.mean(0, keepdims=True), pairs, 0))


def _parts(hq, n):
    """Workgroups that share the streamed rows of a group of 256 resident rows, as the library has it."""
    groups, stages = hq * -(-n // 256), -(-n // 64)
    if groups > 1024:
        return 1
    return min(max(2, 600 // groups, min(1024 // groups, stages // 16)), (stages + 3) // 4)


@pytest.mark.parametrize("hq,n,parts", [(34, 4100, 2), (40, 2000, 2), (12, 2500, 5), (5, 1300, 6), (3, 6200, 8), (1, 4097, 17)])
def test_aggregate_parts(hq, n, parts):
    """Two workgroups to each of 578 groups, and both sides of the rule for fewer; one query head and KV head, repeated."""
    assert parts == _parts(hq, n)
    words = lambda index_heads: vs.aggregate_workspace(hq, hq, index_heads, n)
    assert words(0) >= hq * n * (4 + 16 + 8 * parts)         # row normalisers, fp64 sums, a row sweep's partial results
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(590 + n, 1, 1, n, local=True)
    iv, cv = lists([rng.choice(n, size=n // 10, replace=False)])
    is_, cs = lists([np.unique(np.concatenate([[0], rng.choice(n, size=n // 20, replace=False)]))])
    ref_v, ref_s, ref_r = _oracle(qb, kb, 1, mask=(iv, cv, is_, cs))
    qr, kr = q.repeat(hq, 1, 1).contiguous(), k.repeat(hq, 1, 1).contiguous()
    a_v, a_s, rec = _run(qr, kr, hq, mask=(np.repeat(iv, hq, 0), np.repeat(cv, hq), np.repeat(is_, hq, 0), np.repeat(cs, hq)))
    _close(a_v, np.repeat(ref_v, hq, 0))
    _close(a_s, np.repeat(ref_s, hq, 0))
    assert np.abs(rec - ref_r).max() <= RECALL_ABS


@pytest.mark.parametrize("growth", [6, 12, 100, 300])
@pytest.mark.parametrize("hq,hk,n", [(172, 43, 1473), (8, 2, 1411), (4, 4, 256)])
def test_aggregate_growing_scores(hq, hk, n, growth):
    """Stages without a row maximum, long form, shared out and half groups: the scores of keys n // 4 and n // 2 are 2^(growth / 2) and 2^growth
    above those before them, in every second KV head; with the recall of columns and runs of offsets across whole stages."""
    q, k, v = (x.float() for x in synth.qkv(900 + n, hq, hk, n))
    q[:, :, 0] = 16.0
    k[:, :, 0] = 0.0
    step = growth / (16.0 * 128 ** -0.5 * 1.4426950408889634)
    k[::2, n // 2, 0] = step
    k[::2, n // 4, 0] = 0.5 * step
    q, k = q.bfloat16(), k.bfloat16()
    rng = np.random.default_rng(n)
    mask = [*lists([np.union1d([n // 4], rng.choice(n, 20, replace=False)) for _ in range(hk)]),
            *lists([np.union1d(np.arange(n // 3, n // 3 + 90), rng.choice(n, 9, replace=False)) for _ in range(hk)])]
    a_v, a_s, rec = _run(q.cuda(), k.cuda(), hq, mask=mask)
    group, heads = hq // hk, np.array([0, 1, hq // 2, hq - 1])
    per_q = [m[heads // group] for m in mask]
    ref_v, ref_s, ref_rec = _oracle(synth.to_bits(q)[heads], synth.to_bits(k)[heads // group], 1, mask=per_q)
    _close(a_v[heads], ref_v)
    _close(a_s[heads], ref_s)
    assert np.abs(rec[heads] - ref_rec).max() <= RECALL_ABS


@pytest.mark.parametrize("hq,hk,n", [(1, 1, 127), (3, 1, 128), (4, 2, 129), (1, 1, 200), (8, 2, 255), (3, 3, 256)])
def test_aggregate_half_groups(hq, hk, n):
    """Up to 256 positions of up to 256 heads: the row normalisers come from workgroups of 128 rows."""
    (q, k, v), (qb, kb, vb) = make_qkv(580 + n, hq, hk, n, local=True)
    ref_v, ref_s, _ = _oracle(qb, kb, hq // hk)
    a_v, a_s, _ = _run(q, k, hq)
    _close(a_v, ref_v)
    _close(a_s, ref_s)


@pytest.mark.parametrize("n", [65, 257, 1025, 1100])
def test_aggregate_last_key_nan(n):
    """The last row sees one NaN key, at n = 65, 257 and 1025 the only key of its workgroup's share: its sum, and with it its entry in
    every column and on every diagonal, is NaN whoever adds it up."""
    (q, k, v), _ = make_qkv(570 + n, 1, 1, n, local=True)
    k[:, -1] = float("nan")
    a_v, a_s = torch.zeros(1, n, device="cuda"), torch.zeros(1, n, device="cuda")
    vs.aggregate(q, k, a_v, a_s, torch.empty(vs.aggregate_workspace(1, 1, 0, n), dtype=torch.uint8, device="cuda"))
    assert bool(a_v.isnan().all()) and bool(a_s.isnan().all())


def test_aggregate_8192_one_head_elementwise():
    """n = 8192, one head: 32 groups of resident keys, the streamed rows of each shared out over 18 workgroups (up to 8 stages
    each); every element is compared, together with the recall of a mask."""
    hq, hk, n = 1, 1, 8192
    rng = np.random.default_rng(8192)
    (q, k, v), (qb, kb, vb) = make_qkv(8192, hq, hk, n, local=True)
    sv = [np.concatenate([[0, 1, 2, 3], rng.choice(np.arange(4, n), 200, replace=False)])]
    ss = [np.concatenate([np.arange(64), np.arange(3000, 3040), rng.choice(np.arange(64, n), 30, replace=False)])]
    iv, cv = lists(sv)
    is_, cs = lists(ss)
    a_v, a_s, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    ref_v, ref_s, ref_r = _oracle(qb, kb, 1, mask=(iv, cv, is_, cs))
    _close(a_v, ref_v)
    _close(a_s, ref_s)
    assert np.abs(rec - ref_r).max() <= RECALL_ABS, (rec, ref_r)


def test_aggregate_8192_five_heads_elementwise():
    """The same with five query heads (the same one five times, so that the oracle runs once): 160 groups, six workgroups to a
    group, up to 22 streamed stages each; the 512-entry diagonal rings wrap and every flush window is compared."""
    hq, hk, n = 5, 1, 8192
    rng = np.random.default_rng(8192)
    (q, k, v), (qb, kb, vb) = make_qkv(8192, 1, hk, n, local=True)
    sv = [np.concatenate([[0, 1, 2, 3], rng.choice(np.arange(4, n), 200, replace=False)])]
    ss = [np.concatenate([np.arange(64), np.arange(3000, 3040), rng.choice(np.arange(64, n), 30, replace=False)])]
    iv, cv = lists(sv)
    is_, cs = lists(ss)
    a_v, a_s, rec = _run(q.expand(hq, n, 128).contiguous(), k, hq, mask=(iv, cv, is_, cs))
    ref_v, ref_s, ref_r = _oracle(qb, kb, 1, mask=(iv, cv, is_, cs))
    _close(a_v, np.broadcast_to(ref_v, (hq, n)))
    _close(a_s, np.broadcast_to(ref_s, (hq, n)))
    assert np.abs(rec - ref_r).max() <= RECALL_ABS, (rec, ref_r)


@pytest.mark.parametrize("hq,hk,n", [(32, 8, 1057), (32, 8, 1024), (8, 2, 1000), (1, 1, 4000), (1, 1, 16000)])
def test_aggregate_totals_in_single_precision(hq, hk, n):
    """No systematic error: every head's vectors add up to 1 within 1.5e-7 (a row's normaliser and its entries are rounded by up
    to 2^-20 relative, but at random, which over n rows leaves some 1e-8; the logarithm of a mantissa, rounded towards zero, is
    off by up to 2^-24).  Forms with and without shared-out groups."""
    (q, k, v), _ = make_qkv(540 + n, hq, hk, n, local=True)
    a_v, a_s, _ = _run(q, k, hq)
    assert np.abs(a_v.sum(axis=1) - 1).max() <= 1.5e-7, np.abs(a_v.sum(axis=1) - 1).max()
    assert np.abs(a_s.sum(axis=1) - 1).max() <= 1.5e-7, np.abs(a_s.sum(axis=1) - 1).max()


@pytest.mark.parametrize("hq,hk,n", [(32, 8, 1057), (32, 8, 1024), (8, 2, 1000), (1, 1, 4000), (1, 1, 16000)])
def test_recall_in_single_precision(hq, hk, n):
    """The recall is within 4e-7 of the sum in 64 bits (its shares are single-precision sums over up to 64 tiles, 2^-24 each at
    random), with and without shared-out groups."""
    (q, k, v), _ = make_qkv(540 + n, hq, hk, n, local=True)
    rng = np.random.default_rng(n)
    iv, cv = lists([rng.choice(n, 60, replace=False) for _ in range(hk)])
    is_, cs = lists([np.unique(np.concatenate([np.arange(20), rng.choice(n, 30, replace=False)])) for _ in range(hk)])
    _, _, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    j = torch.arange(n, device="cuda")
    for h in (0, hq - 1):
        g = h // (hq // hk)
        col = torch.zeros(n, dtype=torch.bool, device="cuda")
        off = torch.zeros_like(col)
        col[torch.from_numpy(iv[g, :cv[g]]).cuda().long()] = True
        off[torch.from_numpy(is_[g, :cs[g]]).cuda().long()] = True
        kt, total = k[g].double().t().contiguous(), 0.0
        for a in range(0, n, 1000):
            o = j[a:a + 1000].unsqueeze(1) - j.unsqueeze(0)
            x = (q[h, a:a + 1000].double() @ kt).mul_(128 ** -0.5).masked_fill_(o < 0, -float("inf"))
            total += torch.softmax(x, 1)[(o >= 0) & (col.unsqueeze(0) | off[o.clamp(min=0)])].sum().item()
        assert abs(rec[h] - total / n) <= 4e-7 * total / n, (rec[h], total / n, rec[h] * n / total - 1)


def test_recall_repeated_on_one_workspace():
    """Shared-out groups: the sum and the count of the workgroups' shares start at zero in every call on a workspace, whatever it
    held, and in every replay of a captured call."""
    hq, hk, n = 2, 1, 3000
    (q, k, v), (qb, kb, vb) = make_qkv(77, hq, hk, n, local=True)
    rng = np.random.default_rng(77)
    iv, cv = lists([rng.choice(n, 60, replace=False)])
    is_, cs = lists([np.unique(np.concatenate([np.arange(20), rng.choice(n, 30, replace=False)]))])
    ref_v, _, ref_r = _oracle(qb, kb, hq, mask=(iv, cv, is_, cs))
    dl = _dev_lists(iv, cv, is_, cs)
    ws = torch.full((vs.aggregate_workspace(hq, hk, hk, n),), 0xA5, dtype=torch.uint8, device="cuda")
    a_v, a_s = torch.empty(hq, n, device="cuda"), torch.empty(hq, n, device="cuda")
    rec = torch.empty(hq, device="cuda")
    run = lambda: vs.aggregate(q, k, a_v, a_s, ws, lists=dl, recall=rec)
    for _ in range(3):
        run()
        assert np.abs(rec.cpu().numpy() - ref_r).max() <= 1e-6
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        rec.fill_(float("nan"))
        a_v.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert np.abs(rec.cpu().numpy() - ref_r).max() <= 1e-6
        _close(a_v.cpu().numpy().astype(np.float64), ref_v)


def test_aggregate_group_mean_and_given_lse():
    """out_heads = kv_heads gives the mean over the group's query heads; passing the normalisers of the dense attention
    call instead of recomputing them gives the same vectors."""
    hq, hk, n = 8, 2, 900
    (q, k, v), (qb, kb, vb) = make_qkv(77, hq, hk, n, local=True)
    ref_v, ref_s, _ = _oracle(qb, kb, hq // hk)
    gv = ref_v.reshape(hk, hq // hk, n).mean(axis=1)
    gs = ref_s.reshape(hk, hq // hk, n).mean(axis=1)
    a_v, a_s, _ = _run(q, k, hk)
    _close(a_v, gv)
    _close(a_s, gs)
    o, lse = run_dense(q, k, v)
    b_v, b_s, _ = _run(q, k, hq, lse=lse)
    _close(b_v, ref_v)
    _close(b_s, ref_s)


@pytest.mark.parametrize("hq,hk,n,nv,ns,per_q", [(4, 1, 600, 20, 30, False), (8, 2, 1300, 60, 40, False), (4, 2, 500, 10, 12, True)])
def test_recall_of_a_vertical_slash_mask(hq, hk, n, nv, ns, per_q):
    rng = np.random.default_rng(n)
    (q, k, v), (qb, kb, vb) = make_qkv(400 + n, hq, hk, n, local=True)
    heads = hq if per_q else hk
    sv = [np.concatenate([[0], rng.choice(np.arange(1, n), nv, replace=False)]) for _ in range(heads)]
    ss = [np.concatenate([[0], rng.choice(np.arange(1, n), ns, replace=False)]) for _ in range(heads)]
    iv, cv = lists(sv)
    is_, cs = lists(ss)
    a_v, a_s, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    ref_v, ref_s, ref_r = _oracle(qb, kb, hq // hk, mask=(iv, cv, is_, cs))
    _close(a_v, ref_v)
    _close(a_s, ref_s)
    assert np.abs(rec - ref_r).max() <= RECALL_ABS, (rec, ref_r)
    assert (rec > 0).all() and (rec <= 1 + 1e-5).all()


def test_recall_limits():
    """Every offset selected keeps everything (recall 1); the diagonal alone keeps exactly a_s[0]."""
    hq, hk, n = 4, 1, 400
    (q, k, v), _ = make_qkv(9, hq, hk, n)
    iv, cv = lists([[0]])
    is_, cs = lists([list(range(n))])
    _, _, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    assert np.abs(rec - 1).max() < 1e-4
    iv, cv = lists([[]], cap=1)
    is_, cs = lists([[0]])
    _, a_s, rec = _run(q, k, hq, mask=(iv, cv, is_, cs))
    assert np.abs(rec - a_s[:, 0]).max() < 1e-5


def test_aggregate_argument_errors():
    hq, hk, n = 4, 1, 64
    (q, k, v), _ = make_qkv(1, hq, hk, n)
    a = torch.zeros((hq, n), dtype=torch.float32, device="cuda")
    ws = torch.empty(vs.aggregate_workspace(hq, hk, 0, n), dtype=torch.uint8, device="cuda")
    with pytest.raises(vs.VsError) as e:
        vs.aggregate(q, k, a, a.clone(), ws[:16])
    assert e.value.code == -3
    bad = torch.zeros((3, n), dtype=torch.float32, device="cuda")
    with pytest.raises(vs.VsError) as e:
        vs.aggregate(q, k, bad, bad.clone(), ws)
    assert e.value.code == -2
