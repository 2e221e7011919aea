"""The work that a program using this library gives it, for timing and for comparing two builds.

Shapes follow the benchmark's configurations and the tests: a GQA layer of 32 query and 8 KV heads (8 / 2 and a single
head besides), head_dim 128, 4096 to 131072 positions, the GELU / 256 and the SiLU / 1024 indexer, budgets of the 0.8 to
0.95 cumulative rule or of fixed size.  Inputs are made on the GPU from the seed: keys and values correlated along the
sequence, a few heavy-hitter columns that every query attends to, scores with a near-diagonal band, some long-range bands
and sinks.
"""
import math

import torch

import paper_2603_04460_amd as vs

D = 128
EPS = 1e-30


def listed():
    return [
        # queries of one layer rotated in place before the pipeline, ordinary length
        {"name": "rope_32k", "op": "rope", "heads": 32, "n": 32768, "pos0": 0, "pairing": 0},
        # the paper-shaped indexer alone, long prompt
        {"name": "index_silu1024_64k", "op": "index", "hk": 8, "n": 65536, "d_h": 1024, "act": 0},
        # threshold budget over the longest prompt's scores
        {"name": "select_128k", "op": "select", "heads": 8, "n": 131072, "tau": 0.9, "k_v": 0, "k_s": 0},
        # the whole pipeline of one layer on a short prompt: latency and launches count
        {"name": "layer_4k", "op": "layer", "hq": 32, "hk": 8, "n": 4096, "d_h": 256, "act": 1, "tau": 0.9},
        # the whole pipeline of one layer at the benchmark's length
        {"name": "layer_128k", "op": "layer", "hq": 32, "hk": 8, "n": 131072, "d_h": 256, "act": 1, "tau": 0.9},
        # one head with a small fixed mask of scattered columns and offsets: the smallest attention call
        {"name": "sparse_1head_4k", "op": "sparse", "hq": 1, "hk": 1, "n_q": 4096, "n": 4096, "k_v": 64, "k_s": 128,
         "white": True, "gran": 1},
        # a layer with a fixed budget chosen from structured scores
        {"name": "sparse_32k", "op": "sparse", "hq": 32, "hk": 8, "n_q": 32768, "n": 32768, "k_v": 1024, "k_s": 2048,
         "white": False, "gran": 1},
        # chunked prefill: the last 2000 positions of a prompt of odd length
        {"name": "sparse_chunk_2000", "op": "sparse", "hq": 32, "hk": 8, "n_q": 2000, "n": 50021, "k_v": 1024, "k_s": 1024,
         "white": False, "gran": 1},
        # full attention of a layer, e.g. the layers or lengths that are not made sparse
        {"name": "dense_8k", "op": "dense", "hq": 32, "hk": 8, "n_q": 8192, "n": 8192},
        # full attention of a short chunk against a long context
        {"name": "dense_chunk_500", "op": "dense", "hq": 32, "hk": 8, "n_q": 500, "n": 32768},
        # the distillation target of a layer with the recall of a mask
        {"name": "aggregate_16k", "op": "aggregate", "hq": 32, "hk": 8, "n": 16384, "k_v": 512, "k_s": 512, "recall": True,
         "per_q": False},
        # one training step of the indexer on such a target
        {"name": "train_32k", "op": "train", "hk": 8, "n": 32768, "d_h": 256, "act": 1},
    ]


def _size(rng, lo, hi):
    """Log-uniform, every third a multiple of 1024, the others as they fall (odd ones among them)."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.34:
        n = max(1024, n // 1024 * 1024)
    return max(lo, min(hi, n))


def draw(rng):
    op = rng.choice(["rope", "index", "select", "layer", "sparse", "chunk", "dense", "dense_chunk", "aggregate", "train"])
    hq, hk = rng.choice([(32, 8), (32, 8), (8, 2), (1, 1)])
    width = lambda: rng.choice([(256, 1), (256, 1), (1024, 0), (64, 0), (512, 1)])
    if op == "rope":
        return {"op": op, "heads": rng.choice([32, 8, 1]), "n": _size(rng, 1000, 131072), "pos0": rng.choice([0, 0, 4096]),
                "pairing": rng.choice([0, 1])}
    if op == "index":
        d_h, act = width()
        return {"op": op, "hk": rng.choice([8, 2, 1]), "n": _size(rng, 1000, 131072), "d_h": d_h, "act": act}
    if op == "select":
        n = _size(rng, 1000, 131072)
        fixed = rng.random() < 0.4
        return {"op": op, "heads": rng.choice([8, 8, 32, 1]), "n": n, "tau": 0.0 if fixed else round(rng.uniform(0.8, 0.95), 3),
                "k_v": min(1024, n // 8) if fixed else 0, "k_s": min(2048, n // 8) if fixed else 0}
    if op == "layer":
        d_h, act = width()
        return {"op": op, "hq": hq, "hk": hk, "n": _size(rng, 1000, 65536), "d_h": d_h, "act": act,
                "tau": round(rng.uniform(0.8, 0.95), 3)}
    if op == "sparse":
        n = _size(rng, 1000, 65536)
        return {"op": op, "hq": hq, "hk": hk, "n_q": n, "n": n, "k_v": min(rng.choice([64, 512, 1024]), n // 8),
                "k_s": min(rng.choice([128, 512, 2048]), n // 8), "white": n <= 8192 and rng.random() < 0.3,
                "gran": rng.choice([1, 1, 32])}
    if op == "chunk":
        n = _size(rng, 4096, 131072)
        return {"op": "sparse", "hq": hq, "hk": hk, "n_q": _size(rng, 64, 4096), "n": n, "k_v": min(1024, n // 8),
                "k_s": min(rng.choice([512, 1024]), n // 8), "white": False, "gran": 1}
    if op == "dense":
        n = _size(rng, 500, 16384)
        return {"op": op, "hq": hq, "hk": hk, "n_q": n, "n": n}
    if op == "dense_chunk":
        return {"op": "dense", "hq": hq, "hk": hk, "n_q": _size(rng, 64, 2048), "n": _size(rng, 2048, 65536)}
    if op == "aggregate":
        n = _size(rng, 1000, 16000)
        k = min(512, n // 8)
        return {"op": op, "hq": hq, "hk": hk, "n": n, "k_v": k, "k_s": k, "recall": rng.random() < 0.5, "per_q": rng.random() < 0.3}
    d_h, act = width()
    return {"op": "train", "hk": rng.choice([8, 2, 1]), "n": _size(rng, 1000, 65536 if d_h <= 512 else 32768), "d_h": d_h, "act": act}


# ---- inputs ----
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 9973 + 17)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _tokens(g, heads, n):
    """[heads, n, 128] of unit variance (the first tokens less), neighbouring positions correlated over 33 tokens."""
    x = torch.nn.functional.pad(_normal(g, heads, D, n), (32, 0))
    x = torch.nn.functional.avg_pool1d(x, 33, 1) * math.sqrt(33.0)
    return x.transpose(1, 2).contiguous()


def _hitters(g, heads, n, count=16):
    return torch.randint(0, n, (heads, min(count, n)), generator=g, device="cuda")


def _qkv(g, hq, hk, n_q, n):
    """Rotated q, k and v: 16 columns of every KV head attract all queries."""
    q, k, v = _normal(g, hq, n_q, D), _tokens(g, hk, n), _tokens(g, hk, n)
    u = _normal(g, D)
    u = u / u.norm()
    cols = _hitters(g, hk, n)
    k += 4.0 * u * torch.zeros(hk, n, 1, device="cuda").scatter_(1, cols.unsqueeze(-1), 1.0)
    q += (16.0 / math.sqrt(D)) * u
    return q.bfloat16(), k, v, cols


def _bands(g, heads, n, peak=12.0, count=6, width=None, decay=128.0):
    """Nominal slash logits: a band next to the diagonal and `count` bands at long range."""
    t = torch.arange(n, device="cuda", dtype=torch.float32)
    x = (peak * torch.exp(-t / (n / decay))).repeat(heads, 1)
    c = n * (0.03 + 0.94 * torch.rand(heads, count, generator=g, device="cuda"))
    w = torch.rand(heads, count, generator=g, device="cuda")
    w = (1.0 + w) * (n / 4096.0 if width is None else width / 1.5)
    a = 9.0 + 3.0 * torch.rand(heads, count, generator=g, device="cuda")
    for b in range(count):
        x += a[:, b:b + 1] * torch.exp(-0.5 * ((t - c[:, b:b + 1]) / w[:, b:b + 1]) ** 2)
    return x


def _scores(g, heads, n, white=False, indexer=False):
    """Score vectors [heads, n] for columns and offsets, each a probability distribution; indexer: with the spread of an
    indexer's logits, of which a threshold rule keeps a few percent."""
    l_v, l_s = _normal(g, heads, n), _normal(g, heads, n)
    if indexer:
        l_v = 2.6 * l_v
        l_v[:, :4] += 12.0
        l_v.scatter_add_(1, _hitters(g, heads, n), torch.full((heads, min(16, n)), 9.0, device="cuda"))
        l_s = 2.6 * l_s + _bands(g, heads, n)
    elif not white:
        l_v[:, :4] += 8.0
        l_v.scatter_add_(1, _hitters(g, heads, n), torch.full((heads, min(16, n)), 6.0, device="cuda"))
        l_s = 0.3 * l_s + 0.6 * _bands(g, heads, n, width=48.0, decay=48.0)
    return torch.softmax(l_v.double(), 1).float(), torch.softmax(l_s.double(), 1).float()


def _weights(g, d_h, act):
    uniform = lambda bound, *s: bound * (2.0 * torch.rand(*s, generator=g, device="cuda") - 1.0)
    bd = 14.0 / math.sqrt(d_h)
    W = [uniform(1 / 16.0, 256, d_h), uniform(1 / 16.0, d_h), uniform(bd, d_h), uniform(bd, d_h)]
    return W, vs.IndexerWeights(*W, 0.0, 0.0, act)


def _plant(k, v, W, cols, bands):
    """Moves tokens along the directions of the input that the indexer's two logits follow: bands for the offsets, sinks
    and heavy hitters for the columns."""
    hk, n, _ = k.shape
    d_v = torch.zeros(hk, n, device="cuda")
    d_v[:, :4] = 12.0
    d_v.scatter_(1, cols, 9.0)
    for boost, wd in ((bands, W[3]), (d_v, W[2])):
        d = W[0].double() @ wd.double()
        e = (d / (0.5 * d.dot(d))).float()
        k += boost.unsqueeze(-1) * e[:D]
        v += boost.unsqueeze(-1) * e[D:]


def _bytes(count):
    return torch.empty(max(16, int(count)), dtype=torch.uint8, device="cuda")


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


class _Lists:
    """Budget, output lists and workspace of a selection."""

    def __init__(self, heads, n, tau=0.0, k_v=0, k_s=0):
        sink, local = min(4, n), min(64, n)
        if tau:
            cap = min(n, max(4096, n // 4))
            self.budget = vs.Budget(mode=0, tau_v=tau, tau_s=tau, n_sink=sink, n_local=local, cap_v=cap, cap_s=cap)
        else:
            self.budget = vs.Budget(mode=1, k_v=k_v, k_s=k_s, n_sink=sink, n_local=local, cap_v=k_v + sink, cap_s=k_s + local)
        i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device="cuda")
        self.idx_v, self.idx_s = i32(heads, self.budget.cap_v), i32(heads, self.budget.cap_s)
        self.cnt_v, self.cnt_s, self.status = i32(heads), i32(heads), i32(heads)
        need = vs.select_budget_workspace(heads, n)
        self.ws = _bytes(need) if need else None

    def select(self, a_v, a_s):
        vs.select_budget(a_v, a_s, self.budget, self.idx_v, self.cnt_v, self.idx_s, self.cnt_s, self.status, self.ws)

    def all(self):
        return self.idx_v, self.cnt_v, self.idx_s, self.cnt_s


def prepare(case, seed):
    g, op = _gen(seed), case["op"]
    s = {"case": case}
    if op == "rope":
        s["x"] = _normal(g, case["heads"], case["n"], D).bfloat16()
        return s
    n = case["n"]
    if op in ("index", "layer", "train"):
        hk, d_h = case["hk"], case["d_h"]
        W, s["w"] = _weights(g, d_h, case["act"])
        if op == "layer":
            s["q"], k, v, cols = _qkv(g, case["hq"], hk, n, n)
        else:
            k, v = _tokens(g, hk, n), _tokens(g, hk, n)
            cols = _hitters(g, hk, n)
        _plant(k, v, W, cols, _bands(g, hk, n))
        s["k"], s["v"] = k.bfloat16(), v.bfloat16()
        s["a_v"], s["a_s"] = _f32(hk, n), _f32(hk, n)
        if op == "train":
            s["t_v"], s["t_s"] = _scores(g, hk, n)
            s["loss"] = _f32(1)
            s["grads"] = [_f32(256, d_h), _f32(d_h), _f32(d_h), _f32(d_h)]
            s["ws"] = _bytes(vs.index_train_workspace(hk, n, d_h))
            return s
        s["ws"] = _bytes(vs.index_score_workspace(hk, n, d_h))
        if op == "layer":
            s["lists"] = _Lists(hk, n, tau=case["tau"])
            s["o"] = torch.empty_like(s["q"])
            s["ws_att"] = _bytes(vs.sparse_prefill_workspace(case["hq"], hk, hk, n))
        return s
    if op == "select":
        s["a_v"], s["a_s"] = _scores(g, case["heads"], n, indexer=True)
        s["lists"] = _Lists(case["heads"], n, case["tau"], case["k_v"], case["k_s"])
        return s
    hq, hk = case["hq"], case["hk"]
    n_q = case.get("n_q", n)
    q, k, v, _ = _qkv(g, hq, hk, n_q, n)
    s["q"], s["k"], s["v"] = q, k.bfloat16(), v.bfloat16()
    if op in ("sparse", "aggregate"):
        s["lists"] = _Lists(hk, n, 0.0, case["k_v"], case["k_s"])
        s["lists"].select(*_scores(g, hk, n, case.get("white", False)))
    if op == "aggregate":
        heads = hq if case["per_q"] else hk
        s["a_v"], s["a_s"] = _f32(heads, n), _f32(heads, n)
        s["recall"] = _f32(heads) if case["recall"] else None
        s["ws"] = _bytes(vs.aggregate_workspace(hq, hk, hk if case["recall"] else 0, n))
        return s
    s["o"], s["lse"] = torch.empty_like(q), _f32(hq, n_q)
    if op == "sparse":
        s["ws"] = _bytes(vs.sparse_prefill_workspace(hq, hk, hk, n))
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "rope":
        return vs.rope_apply(s["x"], case["pos0"], 1e6, case["pairing"])
    if op == "index":
        vs.index_score(s["k"], s["v"], s["w"], s["a_v"], s["a_s"], s["ws"])
        return {"a_v": s["a_v"], "a_s": s["a_s"]}
    if op == "select":
        s["lists"].select(s["a_v"], s["a_s"])
        return list(s["lists"].all()) + [s["lists"].status]
    if op == "layer":
        vs.index_score(s["k"], s["v"], s["w"], s["a_v"], s["a_s"], s["ws"])
        s["lists"].select(s["a_v"], s["a_s"])
        vs.sparse_prefill(s["q"], s["k"], s["v"], *s["lists"].all(), s["o"], None, s["ws_att"])
        return {"a_v": s["a_v"], "a_s": s["a_s"], "o": s["o"]}
    if op == "sparse":
        chunk = case["n_q"] != case["n"]
        vs.sparse_prefill(s["q"], s["k"], s["v"], *s["lists"].all(), s["o"], s["lse"], s["ws"],
                          slash_granularity=case["gran"] if case["gran"] != 1 else None,
                          pos0=case["n"] - case["n_q"] if chunk else None)
        return {"o": s["o"], "lse": s["lse"]}
    if op == "dense":
        chunk = case["n_q"] != case["n"]
        vs.dense_prefill(s["q"], s["k"], s["v"], s["o"], s["lse"], pos0=case["n"] - case["n_q"] if chunk else None)
        return {"o": s["o"], "lse": s["lse"]}
    if op == "aggregate":
        vs.aggregate(s["q"], s["k"], s["a_v"], s["a_s"], s["ws"], lists=s["lists"].all() if case["recall"] else None,
                     recall=s["recall"])
        out = {"a_v": s["a_v"], "a_s": s["a_s"]}
        if case["recall"]:
            out["recall"] = s["recall"]
        return out
    vs.index_train_step(s["k"], s["v"], s["w"], s["t_v"], s["t_s"], s["loss"], *s["grads"], s["ws"], eps=EPS)
    return {"loss": s["loss"], "grads": s["grads"]}


# ---- what a pass cannot do without ----
def _indexer_work(hk, n, d_h):
    return hk * n * (512 + 8) + 4 * d_h * 259, 2.0 * (256 + 2) * d_h * hk * n


def _attention_bytes(hq, hk, n_q, n):
    return 256 * (2 * hq * n_q + 2 * hk * n)


def work(case):
    op, n = case["op"], case["n"]
    if op == "rope":
        return {"bytes": 512 * case["heads"] * n, "flops": 6.0 * 64 * case["heads"] * n}
    if op == "select":
        kept = case["heads"] * 4 * (case["k_v"] + case["k_s"])
        return {"bytes": 8 * case["heads"] * n + kept, "flops": 0}
    if op in ("index", "train"):
        b, f = _indexer_work(case["hk"], n, case["d_h"])
        if op == "train":
            # forward, the gradient of W_U and of the down-projections; targets in, gradients out
            return {"bytes": b + 8 * case["hk"] * n + 4 * 259 * case["d_h"], "flops": 2 * f}
        return {"bytes": b, "flops": f}
    hq, hk, n_q = case["hq"], case["hk"], case.get("n_q", n)
    pairs = n_q * (n - n_q) + n_q * (n_q + 1) / 2.0          # causal pairs of a head
    if op == "aggregate":
        # one product of Q and K^T for the normalisers, one for the sums; the lists
        out = (hq if case["per_q"] else hk) * n * 8
        return {"bytes": 256 * (hq + hk) * n + out, "flops": 2.0 * 256 * hq * pairs}
    if op == "dense":
        return {"bytes": _attention_bytes(hq, hk, n_q, n) + 4 * hq * n_q, "flops": 512.0 * hq * pairs}
    if op == "layer":
        b, f = _indexer_work(hk, n, case["d_h"])
        # the recipe keeps 3 to 10 % of the pairs
        return {"bytes": b + 8 * hk * n + _attention_bytes(hq, hk, n, n), "flops": f + 512.0 * hq * 0.05 * pairs}
    kept = min(1.0, (case["k_v"] + case["k_s"]) / float(n)) * pairs
    return {"bytes": _attention_bytes(hq, hk, n_q, n) + 4 * hq * n_q, "flops": 512.0 * hq * kept}


def tolerance(case):
    op = case["op"]
    if op == "select":
        return "exact"
    if op == "rope":
        return {"rel": 2e-3, "max": 0.02}                    # bf16 results; another rounding of a few of them
    if op == "index":
        return {"rel": 5e-5, "max": 2e-3}                    # W_U carries 16 significant bits
    if op == "train":
        return {"rel": 1e-4, "max": 4e-3}                    # sums over all tokens that cancel in part
    if op == "aggregate":
        return {"rel": 1e-5, "max": 4e-4}                    # fp32 sums of exponentials of fp32 scores
    if op == "layer":
        return {"rel": 2e-2, "max": 0.8}                     # bf16 results; an entry at the threshold may change sides
    return {"rel": 1e-2, "max": 0.2}                         # bf16 probabilities and results


# ---- the same in 64 bits ----
def _masks(lists, n):
    """Per index head: columns [n] and offsets [n] that are kept."""
    idx_v, cnt_v, idx_s, cnt_s = lists
    out = []
    for h in range(idx_v.shape[0]):
        pair = []
        for idx, cnt in ((idx_v, cnt_v), (idx_s, cnt_s)):
            m = torch.zeros(n, dtype=torch.bool, device="cuda")
            m[idx[h, :int(cnt[h])].long()] = True
            pair.append(m)
        out.append(pair)
    return out


def _rows(n_q, n):
    """Blocks of query rows, bounded by the scores of a block."""
    step = max(32, min(n_q, (1 << 25) // n))
    return [(a, min(n_q, a + step)) for a in range(0, n_q, step)]


def _keep(i, n, mask):
    off = i.unsqueeze(1) - torch.arange(n, device="cuda").unsqueeze(0)
    keep = off >= 0
    if mask is not None:
        keep &= mask[0].unsqueeze(0) | mask[1][off.clamp(min=0)]
    return keep


def _granular(i, n, mask):
    """Offsets of any row of the aligned 32-row block count for every row of it."""
    first = i // 32 * 32
    last = torch.minimum(first + 31, torch.full_like(first, n - 1))
    reach = torch.cat([torch.zeros(1, dtype=torch.long, device="cuda"), mask[1].long().cumsum(0)])
    j = torch.arange(n, device="cuda").unsqueeze(0)
    hi = (last.unsqueeze(1) - j + 1).clamp(min=0)
    lo = (first.unsqueeze(1) - j).clamp(min=0)
    some = reach[hi] - reach[lo] > 0
    return (i.unsqueeze(1) >= j) & (mask[0].unsqueeze(0) | some)


def _attention64(s, case):
    hq, hk, n_q, n = case["hq"], case["hk"], case["n_q"], case["n"]
    if float(hq) * n_q * n > 1.5e11:
        return None
    masks = _masks(s["lists"].all(), n) if case["op"] == "sparse" else [None] * hk
    o = torch.empty(hq, n_q, D, dtype=torch.float64, device="cuda")
    lse = torch.empty(hq, n_q, dtype=torch.float64, device="cuda")
    for g in range(hk):
        kt, v = s["k"][g].double().t().contiguous(), s["v"][g].double()
        for a, b in _rows(n_q, n):
            i = torch.arange(a, b, device="cuda") + (n - n_q)
            keep = _granular(i, n, masks[g]) if case.get("gran", 1) == 32 else _keep(i, n, masks[g])
            for h in range(g * (hq // hk), (g + 1) * (hq // hk)):
                x = s["q"][h, a:b].double() @ kt
                x.mul_(D ** -0.5).masked_fill_(~keep, -math.inf)
                lse[h, a:b] = torch.logsumexp(x, 1)
                x.sub_(lse[h, a:b].unsqueeze(1)).exp_()
                o[h, a:b] = x @ v
    return {"o": o, "lse": lse}


def _aggregate64(s, case):
    hq, hk, n = case["hq"], case["hk"], case["n"]
    masks = _masks(s["lists"].all(), n) if case["recall"] else None
    a_v = torch.zeros(hq, n, dtype=torch.float64, device="cuda")
    a_s, recall = torch.zeros_like(a_v), torch.zeros(hq, dtype=torch.float64, device="cuda")
    for g in range(hk):
        kt = s["k"][g].double().t().contiguous()
        for a, b in _rows(n, n):
            i, r = torch.arange(a, b, device="cuda"), b - a
            causal = _keep(i, n, None)
            kept = _keep(i, n, masks[g]) if masks else None
            for h in range(g * (hq // hk), (g + 1) * (hq // hk)):
                x = s["q"][h, a:b].double() @ kt
                x = torch.softmax(x.mul_(D ** -0.5).masked_fill_(~causal, -math.inf), 1)
                a_v[h] += x.sum(0)
                if masks:
                    recall[h] += x[kept].sum()
                # rows reversed and moved right by their number: a column then holds one offset
                z = torch.zeros(r, n + r, dtype=torch.float64, device="cuda")
                z[:, :n] = x.flip(1)
                d = z.reshape(-1)[:r * (n + r - 1)].reshape(r, n + r - 1).sum(0)[n - 1 - a:]
                a_s[h, :min(n, d.numel())] += d[:n]
    out = {"a_v": a_v / n, "a_s": a_s / n, "recall": recall / n}
    if not case["per_q"]:
        out = {name: x.reshape(hk, hq // hk, *x.shape[1:]).mean(1) for name, x in out.items()}
    if not case["recall"]:
        del out["recall"]
    return out


def _indexer64(s, case, params):
    """Log-probabilities [hk, n] of the columns and of the offsets."""
    W_U, b_U, W_V, W_S = params
    x = torch.cat([s["k"], s["v"]], 2).double()
    u = x.reshape(-1, 256) @ W_U + b_U
    z = torch.nn.functional.gelu(u) if case["act"] else torch.nn.functional.silu(u)
    shape = s["k"].shape[:2]
    return [torch.log_softmax((z @ w).reshape(shape), 1) for w in (W_V, W_S)]


def exact(case, seed):
    op = case["op"]
    if op == "select":
        return None
    s = prepare(case, seed)
    if op == "rope":
        t = torch.arange(case["n"], device="cuda", dtype=torch.float64) + case["pos0"]
        phi = t.unsqueeze(1) * 1e6 ** (-torch.arange(64, device="cuda", dtype=torch.float64) / 64.0)
        c, w = phi.cos(), phi.sin()
        out = torch.empty(s["x"].shape, dtype=torch.float64, device="cuda")
        ia = torch.arange(64, device="cuda") * (2 if case["pairing"] == 0 else 1)
        ib = ia + (1 if case["pairing"] == 0 else 64)
        for h in range(case["heads"]):
            x = s["x"][h].double()
            out[h][:, ia] = x[:, ia] * c - x[:, ib] * w
            out[h][:, ib] = x[:, ia] * w + x[:, ib] * c
        return out
    if op in ("sparse", "dense"):
        return _attention64(s, case)
    if op == "aggregate":
        return _aggregate64(s, case)
    w = s["w"]
    params = [p.double() for p in (w.W_U, w.b_U, w.W_V, w.W_S)]
    if op == "train":
        for p in params:
            p.requires_grad_(True)
        l_v, l_s = _indexer64(s, case, params)
        loss = sum((l.exp() * (l - t.double().clamp(min=EPS).log())).sum() for l, t in ((l_v, s["t_v"]), (l_s, s["t_s"]))) / case["hk"]
        grads = torch.autograd.grad(loss, params)
        return {"loss": loss.detach().reshape(1), "grads": [x.detach() for x in grads]}
    with torch.no_grad():
        l_v, l_s = _indexer64(s, case, params)
    out = {"a_v": l_v.exp(), "a_s": l_s.exp()}
    if op == "layer":
        out["o"] = None                                      # depends on which entries the rounded scores select
    return out
