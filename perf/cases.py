"""Performance cases of the scoring path, over the range it is used in.

A case is one call that a pre-ranking server makes: scoring a batch of
requests (``ColdModel.score``, or the call prepared once with
``ColdModel.prepare`` where a server reuses its buffers), or picking each
request's best rows by eCPM afterwards (``select_topn``).  The models are the
repository's own configurations (``synth.CONFIGS``); sizes run from the
smallest single request to the largest batch.

``listed`` gives the named cases, ``draw`` more of the same ranges,
``prepare`` a case's inputs and handles, ``run`` one pass, ``work`` the bytes
and operations a pass cannot do without, ``tolerance`` what another correct
implementation at the same precision may differ by, ``exact`` the outputs in
64 bits.
"""
import math
import random

import numpy as np
import torch

from paper_2007_16122_amd import binding, synth

DEV = "cuda"
TORCH_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

# every field of a scoring case and its value where a case does not give one
SCORE_DEFAULTS = dict(
    kind="score", base="serving_bf16", requests=1, ads=2000, ragged=False,
    vocab=1_000_000, dtype="bf16", hashed=False, linear_log=False, topk=0,
    literal_se=False, gpu_cross=False, importance=False, prepared=False, narrow=False,
    n_user=12, n_seq=0, n_ad=24, n_cross=12, emb_dim=16)


def _score(**kw):
    case = dict(SCORE_DEFAULTS)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest call: one request of the fp32 model, launch-bound
        _score(name="tiny_fp32_one_request", base="tiny_fp32", ads=512, dtype="f32",
               vocab=10_000, n_user=4, n_ad=8, n_cross=4, emb_dim=8, prepared=True),
        # online serving at low load: one request of 2,000 ads, latency
        _score(name="serving_bf16_one_request", prepared=True),
        # the request queue of a moment gathered into one call: uneven sizes
        # (one request without candidates), SE weights asked for
        _score(name="serving_bf16_ragged_7", requests=7, ads=1111, ragged=True, importance=True),
        # serving at full load: 32 requests of 2,000 ads
        _score(name="serving_bf16_batch_32", requests=32),
        # the model with behaviour sequences, one request and a full batch
        _score(name="multivalued_f16_one_request", base="multivalued_fp16_ll", dtype="f16",
               linear_log=True, n_seq=6, prepared=True),
        _score(name="multivalued_f16_batch_32", base="multivalued_fp16_ll", dtype="f16",
               linear_log=True, n_seq=6, requests=32),
        # the largest: 128 requests of 10,000 ads on hashed 10M-row tables
        _score(name="large_f16_batch_128", base="large_fp16_ll", dtype="f16", linear_log=True,
               hashed=True, vocab=10_000_000, n_user=16, n_ad=32, n_cross=16,
               requests=128, ads=10_000),
        # feature-group selection: 200 groups of which a request keeps 100,
        # one request with its importance and mask, and an uneven batch
        _score(name="wide_topk_bf16_one_request", base="wide_prune_bf16", n_user=50, n_ad=100,
               n_cross=50, topk=100, ads=5000, importance=True, prepared=True),
        _score(name="wide_topk_bf16_ragged_6", base="wide_prune_bf16", n_user=50, n_ad=100,
               n_cross=50, topk=100, requests=6, ads=1501, ragged=True),
        # Eq. 2 as printed: one fully connected SE layer
        _score(name="literal_se_bf16_batch_32", requests=32, literal_se=True),
        # raw 64-bit ids, cross features formed on the GPU, odd sizes
        _score(name="gpu_cross_hashed_f16_11", base="serving_bf16", dtype="f16", linear_log=True,
               hashed=True, gpu_cross=True, requests=11, ads=1999, n_user=11, n_ad=23, n_cross=13),
        # the step after scoring: the best 200 of every request by eCPM
        dict(name="topn_batch_32", kind="topn", requests=32, ads=2000, ragged=False, n_top=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(("tiny", "serving", "serving", "serving", "multivalued", "multivalued",
                       "large", "wide", "literal", "topn"))
    ragged = rng.random() < 0.5
    if what == "topn":
        return dict(kind="topn", requests=_log_int(rng, 1, 128), ads=_log_int(rng, 50, 10_000),
                    ragged=ragged, n_top=_log_int(rng, 1, 1024))
    case = _score(ragged=ragged, importance=rng.random() < 0.25, prepared=rng.random() < 0.5)
    if what == "tiny":
        case.update(base="tiny_fp32", dtype="f32", requests=_log_int(rng, 1, 8),
                    ads=_log_int(rng, 32, 4096), vocab=_log_int(rng, 1000, 100_000),
                    n_user=rng.randint(2, 8), n_ad=rng.randint(4, 16), n_cross=rng.randint(2, 8),
                    emb_dim=8)
        return case
    case.update(requests=_log_int(rng, 1, 64), ads=_log_int(rng, 50, 4000),
                vocab=_log_int(rng, 10_000, 1_000_000), dtype=rng.choice(("bf16", "f16")),
                hashed=rng.random() < 0.4, linear_log=rng.random() < 0.4,
                gpu_cross=rng.random() < 0.2, narrow=rng.random() < 0.15,
                n_user=rng.randint(6, 16), n_ad=rng.randint(12, 32), n_cross=rng.randint(6, 16),
                emb_dim=rng.choice((16, 16, 16, 16, 8, 32)))
    if what == "multivalued":
        case.update(base="multivalued_fp16_ll", dtype="f16", linear_log=True,
                    n_seq=rng.randint(1, 8), requests=_log_int(rng, 1, 40))
    elif what == "large":
        case.update(base="large_fp16_ll", dtype="f16", linear_log=True, hashed=True,
                    requests=rng.randint(24, 100), ads=_log_int(rng, 2000, 8000),
                    vocab=_log_int(rng, 1_000_000, 5_000_000), emb_dim=16, narrow=False)
    elif what == "wide":
        m4 = rng.randint(25, 50)
        case.update(base="wide_prune_bf16", n_user=m4, n_ad=2 * m4, n_cross=m4 + rng.randint(-3, 0),
                    requests=_log_int(rng, 1, 8), ads=_log_int(rng, 200, 5000), emb_dim=16,
                    gpu_cross=False, narrow=False)
        m = case["n_user"] + case["n_ad"] + case["n_cross"]
        case.update(topk=int(m * rng.uniform(0.3, 0.7)))
    elif what == "literal":
        case.update(literal_se=True, requests=_log_int(rng, 1, 40))
    return case


# ------------------------------------------------------------------ inputs
def _counts(case):
    """Candidates of every request: a function of the case alone."""
    q, ads = case["requests"], case["ads"]
    if not case["ragged"] or q == 1:
        return [ads] * q
    rng = random.Random(f"{q} x {ads}")
    w = [math.exp(rng.gauss(0.0, 0.7)) for _ in range(q)]
    if q >= 4:
        w[1] = 0.0          # a request without candidates
    total = q * ads
    c = [int(total * x / sum(w)) for x in w]
    c[-1] += total - sum(c)
    return c


def _offsets(case):
    off = np.zeros(case["requests"] + 1, np.int32)
    off[1:] = np.cumsum(_counts(case))
    return off


def _config(case):
    pairs = ()
    if case["gpu_cross"]:
        pairs = tuple((f % case["n_user"], f % case["n_ad"]) for f in range(case["n_cross"]))
    over = dict(
        n_requests=case["requests"], cand_per_request=case["ads"], n_user=case["n_user"],
        n_seq=case["n_seq"], n_ad=case["n_ad"], n_cross=case["n_cross"], emb_dim=case["emb_dim"],
        vocab=case["vocab"], dtype=case["dtype"], hashed=case["hashed"],
        linear_log=case["linear_log"], topk_k=case["topk"], cross_pairs=pairs,
        se_form="literal" if case["literal_se"] else "squeeze")
    if case["narrow"]:      # a lighter network: the paper's without its widest layer
        m = case["n_user"] + case["n_seq"] + case["n_ad"] + case["n_cross"]
        over["widths"] = (m * case["emb_dim"], 512, 256, 128, 64, 2)
    return synth.config(case["base"], **over)


def _cdf(n, s):
    c = torch.cumsum(torch.arange(1, n + 1, dtype=torch.float64, device=DEV) ** (-s), 0)
    return c / c[-1]


def _ids(gen, host, cfg, cdf, size):
    """Ids of one field: Zipf ranks, the hot ones scattered over the table
    (direct ids) or over the 64-bit raw ids (hashed; as int64 bit patterns)."""
    u = torch.rand(size, dtype=torch.float64, device=DEV, generator=gen)
    rank = torch.searchsorted(cdf, u, right=True).clamp_(max=cfg.vocab - 1)
    if cfg.hashed:
        return rank * (2 * host.getrandbits(61) + 1) + host.getrandbits(62)
    a = next(x for x in iter(lambda: host.randrange(1, cfg.vocab), None)
             if math.gcd(x, cfg.vocab) == 1)
    return ((rank * a + host.randrange(cfg.vocab)) % cfg.vocab).to(torch.int32)


def _inputs(case, seed):
    """Tables, parameters and one batch, on the GPU."""
    cfg = _config(case)
    gen = torch.Generator(device=DEV).manual_seed(7 + 1000003 * seed)
    host = random.Random(1 + 1000003 * seed)
    dt = TORCH_DTYPE[cfg.dtype]
    tables = []
    for g in range(cfg.n_groups):
        t = torch.empty((cfg.vocab, cfg.emb_dim), dtype=dt, device=DEV)
        if cfg.table_scheme(g) == "big":    # large-valued behaviour features: pools pass 65504
            t.random_(-1024, 1024, generator=gen)
            t.mul_(16)
        else:
            t.normal_(0.0, 0.05, generator=gen)
        tables.append(t)
    params = binding.params_to_device(synth.make_params(cfg, seed=cfg.seed + 17 * seed), cfg.dtype, DEV)
    cdf = _cdf(cfg.vocab, cfg.zipf_s)
    off = _offsets(case)
    q, r = case["requests"], int(off[-1])

    def columns(n, size):
        dt_id = torch.int64 if cfg.hashed else torch.int32
        if n == 0 or size == 0:
            return torch.zeros(1, dtype=dt_id, device=DEV)
        return torch.stack([_ids(gen, host, cfg, cdf, size) for _ in range(n)])

    seq_off = np.zeros(cfg.n_seq * q + 1, np.int32)
    lens = np.random.default_rng(seed).integers(1, cfg.seq_len_max + 1, cfg.n_seq * q)
    seq_off[1:] = np.cumsum(lens)
    batch = dict(
        req_off=torch.from_numpy(off).to(DEV), user_ids=columns(cfg.n_user, q),
        ad_ids=columns(cfg.n_ad, r),
        cross_ids=columns(0 if cfg.cross_pairs else cfg.n_cross, r),
        seq_off=torch.from_numpy(seq_off).to(DEV),
        seq_ids=torch.cat([_ids(gen, host, cfg, cdf, int(seq_off[(f + 1) * q] - seq_off[f * q]))
                           for f in range(cfg.n_seq)]) if cfg.n_seq else None,
        n_rows=r)
    return cfg, tables, params, batch


def _topn_inputs(case, seed):
    off = _offsets(case)
    r = int(off[-1])
    gen = torch.Generator(device=DEV).manual_seed(11 + 1000003 * seed)
    scores = torch.sigmoid(torch.randn(r, device=DEV, generator=gen) * 0.8 - 2.0)
    bids = torch.from_numpy(synth.make_bids(synth.CONFIGS["serving_bf16"], r, seed=seed)).to(DEV)
    return scores, bids, torch.from_numpy(off).to(DEV)


def prepare(case, seed):
    if case["kind"] == "topn":
        scores, bids, off = _topn_inputs(case, seed)
        return dict(case=case, scores=scores, bids=bids, off=off)
    cfg, tables, params, batch = _inputs(case, seed)
    model = binding.ColdModel(cfg, device=DEV)
    model.load(tables, params)
    r, q = batch["n_rows"], case["requests"]
    model.ensure_workspace(r, q)
    imp = torch.empty((r, cfg.n_groups), dtype=torch.float32, device=DEV) if case["importance"] else None
    mask = torch.empty((q, cfg.n_groups), dtype=torch.uint8, device=DEV) \
        if case["importance"] and cfg.topk_k else None
    st = dict(case=case, model=model, batch=batch, imp=imp, mask=mask, call=None)
    if case["prepared"]:
        scores = torch.empty(r, dtype=torch.float32, device=DEV)
        st["call"] = model.prepare(batch, scores, importance=imp, group_mask=mask)
    return st


def run(state):
    if state["case"]["kind"] == "topn":
        return list(binding.select_topn(state["scores"], state["bids"], state["off"],
                                        state["case"]["n_top"]))
    if state["call"] is not None:
        scores = state["call"]()
    else:
        scores = state["model"].score(state["batch"], importance=state["imp"],
                                      group_mask=state["mask"])
    return [t for t in (scores, state["imp"], state["mask"]) if t is not None]


# ------------------------------------------------------------ work, tolerance
def _distinct(n, vocab, s):
    """Expected number of distinct rows among n Zipf(s) draws from vocab."""
    if n <= 0:
        return 0.0
    head = np.arange(1, min(vocab, 1000) + 1, dtype=np.float64)
    edges = np.unique(np.rint(np.geomspace(1000, max(vocab, 1001), 400)))
    mid, width = 0.5 * (edges[1:] + edges[:-1]) + 0.5, edges[1:] - edges[:-1]
    k = np.concatenate([head, mid]) if vocab > 1000 else head
    w = np.concatenate([np.ones_like(head), width]) if vocab > 1000 else np.ones_like(head)
    p = k ** (-s)
    p = p / (p * w).sum()
    return float((w * -np.expm1(n * np.log1p(-np.minimum(p, 1 - 1e-12)))).sum())


def work(case):
    off = _offsets(case)
    q, r = case["requests"], int(off[-1])
    if case["kind"] == "topn":
        return {"bytes": 8 * r + 4 * (q + 1) + 8 * q * case["n_top"], "flops": r}
    cfg = _config(case)
    es = 4 if cfg.dtype == "f32" else 2
    ib = 8 if cfg.hashed else 4
    row = cfg.emb_dim * es
    m = cfg.n_groups
    fields = cfg.n_ad + cfg.n_cross
    pooled = cfg.n_seq * q * (cfg.seq_len_max + 1) // 2
    by = 4 * (q + 1) + cfg.n_user * q * ib + pooled * (ib + 4)
    by += (cfg.n_ad + (0 if cfg.cross_pairs else cfg.n_cross)) * r * ib
    by += row * (fields * _distinct(r, cfg.vocab, cfg.zipf_s)
                 + cfg.n_user * _distinct(q, cfg.vocab, cfg.zipf_s)
                 + cfg.n_seq * _distinct(pooled // max(cfg.n_seq, 1), cfg.vocab, cfg.zipf_s))
    w = list(cfg.widths)
    by += sum(es * a * b + 4 * b for a, b in zip(w[:-1], w[1:]))
    se = 4 * m * cfg.d_in if case["literal_se"] else 8 * m * cfg.se_hidden
    by += se + 4 * r + (4 * r * m if case["importance"] else 0)
    if cfg.topk_k:                       # the first layer sees the kept groups
        w[0] = min(cfg.topk_k, m) * cfg.emb_dim
    flops = 2 * r * sum(a * b for a, b in zip(w[:-1], w[1:]))
    flops += 2 * r * (m * cfg.d_in if case["literal_se"] else 2 * m * cfg.se_hidden)
    flops += 3 * r * m * cfg.emb_dim     # squeeze and reweighting
    return {"bytes": int(by), "flops": int(flops)}


def tolerance(case):
    if case["kind"] == "topn":
        return "exact"
    # about four times the distance to exact() that the path shows
    rel = {"f32": 2e-7, "bf16": 6e-3, "f16": 2e-3}[case["dtype"]]
    tol = {"rel": rel, "max": 10 * rel}
    if case["topk"]:
        tol["differ"] = 0.005            # groups tied in importance to fp32 rounding
    return tol


# ----------------------------------------------------------------- 64 bits
def _mix64(z):
    """SplitMix64's output function on int64 bit patterns."""
    def shr(x, n):
        return (x >> n) & ((1 << (64 - n)) - 1)

    def c(v):
        return v - (1 << 64) if v >= 1 << 63 else v
    z = (z ^ shr(z, 30)) * c(0xbf58476d1ce4e5b9)
    z = (z ^ shr(z, 27)) * c(0x94d049bb133111eb)
    return z ^ shr(z, 31)


def _umod(h, n):
    """Unsigned h mod n for int64 bit patterns, n < 2^31."""
    half = (h >> 1) & 0x7FFFFFFFFFFFFFFF
    return ((half % n) * 2 + (h & 1)) % n


def _hash_rows(raw, g, n):
    salt = ((g + 1) * 0x9e3779b97f4a7c15) & 0xFFFFFFFFFFFFFFFF
    return _umod(_mix64(raw ^ (salt - (1 << 64) if salt >= 1 << 63 else salt)), n)


def _exact_topn(case, seed):
    scores, bids, off = (t.cpu().numpy() for t in _topn_inputs(case, seed))
    n = case["n_top"]
    ecpm = scores * bids                 # one fp32 product, by definition
    rows = np.full((case["requests"], n), -1, np.int32)
    top = np.full((case["requests"], n), -np.inf, np.float32)
    for i in range(case["requests"]):
        e = ecpm[off[i]:off[i + 1]]
        k = np.argsort(-e, kind="stable")[:n]
        rows[i, :len(k)] = k + off[i]
        top[i, :len(k)] = e[k]
    return [rows, top]


def exact(case, seed):
    if case["kind"] == "topn":
        return _exact_topn(case, seed)
    cfg, tables, params, batch = _inputs(case, seed)
    f64 = torch.float64
    off = _offsets(case)
    q, r = case["requests"], int(off[-1])
    p = {k: ([t.to(f64) for t in v] if isinstance(v, list) else v.to(f64)) for k, v in params.items()}
    req = torch.repeat_interleave(torch.arange(q, device=DEV),
                                  torch.from_numpy(np.diff(off).astype(np.int64)).to(DEV))
    nu, ns, na, nx = cfg.n_user, cfg.n_seq, cfg.n_ad, cfg.n_cross
    m, d = cfg.n_groups, cfg.emb_dim

    def rows_of(ids, g):
        return _hash_rows(ids, g, cfg.vocab) if cfg.hashed else ids.long()

    user = [tables[f][rows_of(batch["user_ids"][f], f)].to(f64) for f in range(nu)]
    pooled = []
    so = batch["seq_off"].long()
    for f in range(ns):
        lo, hi = int(so[f * q]), int(so[(f + 1) * q])
        e = tables[nu + f][rows_of(batch["seq_ids"][lo:hi], nu + f)].to(f64)
        lens = so[f * q + 1:(f + 1) * q + 1] - so[f * q:(f + 1) * q]
        seg = torch.repeat_interleave(torch.arange(q, device=DEV), lens)
        pooled.append(torch.zeros((q, d), dtype=f64, device=DEV).index_add_(0, seg, e))

    def embed(lo, hi):
        qq = req[lo:hi]
        out = [t[qq] for t in user] + [t[qq] for t in pooled]
        for f in range(na):
            g = nu + ns + f
            out.append(tables[g][rows_of(batch["ad_ids"][f][lo:hi], g)].to(f64))
        for f in range(nx):
            g = nu + ns + na + f
            if cfg.cross_pairs:
                u, a = cfg.cross_pairs[f]
                uid, aid = batch["user_ids"][u][qq].long(), batch["ad_ids"][a][lo:hi].long()
                row = _hash_rows(_mix64(uid) ^ aid, g, cfg.vocab)
            else:
                row = rows_of(batch["cross_ids"][f][lo:hi], g)
            out.append(tables[g][row].to(f64))
        return torch.stack(out, 1)       # [rows][m][d]

    def weights(e):
        if case["literal_se"]:
            return torch.sigmoid(e.reshape(len(e), m * d) @ p["se_w1"].T + p["se_b1"])
        h = torch.relu(e.mean(2) @ p["se_w1"].T + p["se_b1"])
        return torch.sigmoid(h @ p["se_w2"].T + p["se_b2"])

    step = max(1, (1 << 25) // (m * d))
    spans = [(lo, min(r, lo + step)) for lo in range(0, r, step)]
    keep_s = case["importance"] or cfg.topk_k
    s_all = torch.cat([weights(embed(lo, hi)) for lo, hi in spans]) if keep_s else None
    mask = None
    if cfg.topk_k:
        total = torch.zeros((q, m), dtype=f64, device=DEV).index_add_(0, req, s_all)
        order = torch.sort(total, dim=1, descending=True, stable=True).indices[:, :cfg.topk_k]
        mask = torch.zeros((q, m), dtype=f64, device=DEV).scatter_(1, order, 1.0)
    scores = []
    for lo, hi in spans:
        e = embed(lo, hi)
        s = s_all[lo:hi] if keep_s else weights(e)
        if mask is not None:
            s = s * mask[req[lo:hi]]
        x = (e * s[:, :, None]).reshape(hi - lo, m * d)
        if cfg.linear_log:
            x = torch.where(x.abs() <= 1, x, torch.sign(x) * (torch.log(x.abs().clamp(min=1)) + 1))
        for w, b in zip(p["mlp_w"][:-1], p["mlp_b"][:-1]):
            x = torch.relu(x @ w.T + b)
        z = x @ p["mlp_w"][-1].T + p["mlp_b"][-1]
        scores.append(torch.sigmoid(z[:, 0]) if z.shape[1] == 1 else torch.sigmoid(z[:, 1] - z[:, 0]))
    out = [torch.cat(scores)]
    if case["importance"]:
        out.append(s_all)
        if mask is not None:
            out.append(mask.to(torch.uint8))
    return out
