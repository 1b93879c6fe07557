"""Workloads whose time is watched: searches through the public binding.

A case names a corpus (documents, centroids, document lengths, how evenly the
centroids are used, code bits), a batch of queries (how many, tokens each,
element type) and the search's knobs.  The corpora follow the recipes of
``synth.configs`` (unit vectors around random unit centroids, noise 0.05;
queries are noised copies of a document's tokens, noise 0.1), drawn on the
GPU so that an index is there in seconds.

A retrieval service loads its index once and answers query after query, so
a corpus is built once per process and kept; the seed of a case decides its
queries.  The residual quantiser is fixed on a sample of the tokens.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_23553_amd import Builder, chimera

DIM = 128
CHUNK_TOKENS = 2_000_000   # tokens generated and indexed at a time
SAMPLE_TOKENS = 2_000_000  # tokens that fix the quantiser
SOURCES = 8192             # documents that queries are drawn from
KEEP_TOKENS = 420_000_000  # indexed tokens kept by one process

FIXED, LOGNORMAL, UNIFORM = "fixed", "lognormal", "uniform"


def _case(name, *, ndocs, ncent, nbits=2, lens=LOGNORMAL, len_mean=64, zipf=False, deleted=0.0, rabitq=False,
          call="search", nq, Tq=32, dtype="bf16", nprobe, ncand, k, kfb=0, chunks=0):
    c = dict(ndocs=ndocs, ncent=ncent, nbits=nbits, lens=lens, len_mean=len_mean, zipf=zipf, deleted=deleted,
             rabitq=rabitq, call=call, nq=nq, Tq=Tq, dtype=dtype, nprobe=nprobe, ncand=ncand, k=k, kfb=kfb,
             chunks=chunks)
    return dict(c, name=name) if name else c


def listed():
    small = dict(ndocs=100_000, ncent=16_384, nprobe=4, ncand=4096, k=10)
    shard = dict(ndocs=2_200_000, ncent=262_144, len_mean=70, zipf=True, nprobe=16, ncand=16_384, k=100)
    return [
        # a unit-test sized collection, queries as the encoder gives them (float32)
        _case("tiny-f32", ndocs=1000, ncent=1024, lens=FIXED, len_mean=32, nq=16, dtype="f32", nprobe=2, ncand=256,
              k=10),
        # one user's query against a collection of LoTTE's size: latency
        _case("100k-one", nq=1, **small),
        # an offline batch against the same collection
        _case("100k-batch", nq=256, **small),
        # the same collection, candidates refined from their tokens' own scores
        _case("100k-refine", call="refine", nq=64, **small),
        # the same collection, the best candidates rescored by the host in full precision
        _case("100k-collab", call="collab", nq=64, kfb=40, chunks=4, **small),
        # a collection with odd sizes everywhere, short float32 queries, a tenth of its documents deleted
        _case("ragged-deleted", ndocs=30_011, ncent=5_003, len_mean=41, deleted=0.1, nq=77, Tq=21, dtype="f32",
              nprobe=7, ncand=3_001, k=37),
        # the paper's code split: 1-bit RaBitQ codes scored on the GPU
        _case("rabitq-batch", ndocs=20_000, ncent=8_192, rabitq=True, call="rabitq", nq=256, nprobe=4, ncand=4096,
              k=10),
        # a million passages whose topics are unevenly popular, a full batch
        _case("1m-batch", ndocs=1_000_000, ncent=65_536, len_mean=70, zipf=True, nq=1024, nprobe=8, ncand=8192, k=100),
        # one of four document-range shards of a collection of MS MARCO's size: one query, and a batch
        _case("shard-one", nq=1, **shard),
        _case("shard-batch", nq=1024, **shard),
        # long documents, 4-bit codes, 64 query tokens, deep results
        _case("long-batch", ndocs=250_000, ncent=65_536, nbits=4, lens=UNIFORM, len_mean=320, nq=128, Tq=64,
              nprobe=32, ncand=32_768, k=1000),
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(c):
    """Rough cost of a pass: documents walked, tokens scored, centroids compared."""
    blocks = 1 if c["Tq"] <= 32 else 2
    per = 0.3 * c["ndocs"] * (1 + c["nprobe"] / 8) + blocks * (c["ncand"] * c["len_mean"] + c["ncent"])
    return c["nq"] * per * (20 if c["call"] == "refine" else 4 if c["call"] != "search" else 1)


def draw(rng):
    call = rng.choice(["search"] * 7 + ["refine", "collab", "rabitq"])
    lens = rng.choice([FIXED, LOGNORMAL, LOGNORMAL, LOGNORMAL, UNIFORM])
    mean = {FIXED: 32, LOGNORMAL: rng.randint(40, 80), UNIFORM: 320}[lens]
    most = 1_000_000 if lens == LOGNORMAL else 200_000
    if call == "rabitq":
        lens, mean, most = LOGNORMAL, rng.randint(40, 70), 20_000
    elif call != "search":
        most = 100_000
    ndocs = _spread(rng, 1000, most)
    ntok = ndocs * mean
    ncent = _spread(rng, max(512, int(2 * math.sqrt(ntok))), max(1024, int(16 * math.sqrt(ntok))))
    Tq = rng.choice([32, 32, 32, rng.randint(4, 31), rng.randint(33, 64), 64])
    nprobe = _spread(rng, 1, 32)
    ncand = _spread(rng, 64, 32_768)
    # enough documents in the probed lists for the asked results
    found = min(ndocs, ncand, int(0.2 * Tq * nprobe * ntok / ncent) + 1)
    k = min(_spread(rng, 1, 1000), max(1, found // 2))
    kfb = chunks = 0
    if call == "collab":
        k = min(k, 50)
        kfb, chunks = k * rng.randint(2, 4), rng.choice([1, 2, 4, 5])
        ncand = max(ncand, kfb)
    c = _case(None, ndocs=ndocs, ncent=ncent, nbits=rng.choice([2, 2, 4]), lens=lens, len_mean=mean,
              zipf=rng.random() < 0.4, deleted=rng.choice([0.0, 0.0, 0.0, 0.15]), rabitq=call == "rabitq", call=call,
              nq=_spread(rng, 1, 1024), Tq=Tq, dtype=rng.choice(["bf16", "bf16", "f32"]), nprobe=nprobe,
              ncand=ncand, k=k, kfb=kfb, chunks=chunks)
    top = 0.5 * max(_cost(x) for x in listed())
    c["nq"] = max(1, min(c["nq"], int(top / (_cost(c) / c["nq"]))))
    return c


# ------------------------------------------------------------ inputs
def _gen(*key):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence(key).generate_state(1, np.uint64)[0] >> 1))
    return g


def _grid(x):
    """The nearest multiple of 2^-11 that bfloat16 holds (ties to even)."""
    return torch.where(x.abs() < 0.0625, torch.round(x * 2048) / 2048, x.to(torch.bfloat16).float())


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


_CORPUS_KEYS = ("ndocs", "ncent", "nbits", "lens", "len_mean", "zipf", "deleted", "rabitq")


class _Corpus:
    """Documents of one collection: their lengths, centroids, and their tokens chunk by chunk."""

    def __init__(self, spec):
        self.spec = spec
        self.seed = (spec["ndocs"], spec["ncent"], spec["len_mean"], int(spec["zipf"]))
        rng = np.random.default_rng(self.seed)
        n, mean = spec["ndocs"], spec["len_mean"]
        if spec["lens"] == FIXED:
            lens = np.full(n, mean)
        elif spec["lens"] == LOGNORMAL:
            lens = np.clip(np.rint(rng.lognormal(math.log(mean) - 0.125, 0.5, n)), 8, 180)
        else:
            lens = rng.integers(mean * 2 // 5, mean * 8 // 5 + 1, n)
        self.lens = lens.astype(np.int32)
        self.off = np.zeros(n + 1, np.int64)
        np.cumsum(self.lens, out=self.off[1:])
        self.ntok = int(self.off[-1])
        self.cent = _grid(_unit(torch.randn(spec["ncent"], DIM, generator=_gen(*self.seed, 1), device="cuda")))
        self.cdf = None
        if spec["zipf"]:
            w = torch.arange(1, spec["ncent"] + 1, device="cuda", dtype=torch.float64) ** -1.1
            self.cdf = torch.cumsum(w / w.sum(), 0)
            self.perm = torch.randperm(spec["ncent"], generator=_gen(*self.seed, 2), device="cuda")
        self.deleted = rng.choice(n, int(n * spec["deleted"]), replace=False) if spec["deleted"] else None
        self.signs = np.where(rng.random(DIM) < 0.5, -1, 1).astype(np.int8)

    def chunks(self):
        """(first document, last document + 1, tokens bf16 [rows, DIM], centroids int32 [rows]) on the GPU."""
        d0 = i = 0
        n = self.spec["ndocs"]
        while d0 < n:
            d1 = max(d0 + 1, int(np.searchsorted(self.off, self.off[d0] + CHUNK_TOKENS, side="right")) - 1)
            rows = int(self.off[d1] - self.off[d0])
            g = _gen(*self.seed, 3, i)
            if self.cdf is None:
                cid = torch.randint(self.spec["ncent"], (rows,), generator=g, device="cuda")
            else:
                u = torch.rand(rows, generator=g, device="cuda", dtype=torch.float64)
                cid = self.perm[torch.searchsorted(self.cdf, u).clamp_(max=self.spec["ncent"] - 1)]
            tok = _grid(_unit(self.cent[cid] + 0.05 * torch.randn(rows, DIM, generator=g, device="cuda")))
            yield d0, d1, tok.to(torch.bfloat16), cid.int()
            d0, i = d1, i + 1

    def index(self, fullbit):
        """The device index, and the tokens of the documents that queries are drawn from."""
        def host(t):
            return t.view(torch.int16).cpu().numpy().view(np.uint16)

        b = Builder(host(self.cent.to(torch.bfloat16)), self.spec["nbits"])
        if self.spec["rabitq"]:
            b.rabitq(self.signs)
        step = max(1, self.spec["ndocs"] // SOURCES)
        pool, docs, store = [], [], []
        for d0, d1, tok, cid in self.chunks():
            bits, ids = host(tok), cid.cpu().numpy()
            if d0 == 0:
                b.add_residuals(bits[:SAMPLE_TOKENS], ids[:SAMPLE_TOKENS])
                b.freeze()
                b.reserve(self.spec["ndocs"], self.ntok)
            b.add_docs(bits, ids, self.lens[d0:d1])
            src = np.arange(-(-d0 // step) * step, d1, step)
            rows = np.concatenate([np.arange(self.off[d], self.off[d + 1]) for d in src] or [np.empty(0, np.int64)])
            pool.append(tok[torch.from_numpy(rows - self.off[d0]).cuda()])
            docs.append(src)
            if fullbit:
                store.append(bits)
        idx = b.upload(0)
        b.close()
        if fullbit:
            idx.attach_fullbit(np.concatenate(store))
        if self.deleted is not None:
            idx.delete(self.deleted)
        n = self.lens[np.concatenate(docs)].astype(np.int64)
        return idx, torch.cat(pool), torch.from_numpy(n).cuda(), torch.from_numpy(np.cumsum(n) - n).cuda()

    def queries(self, built, case, seed):
        _, pool, n, beg = built
        nq, Tq = case["nq"], case["Tq"]
        g = _gen(*self.seed, 4, seed)
        d = torch.randint(len(n), (nq, 1), generator=g, device="cuda")
        v = pool[beg[d] + torch.arange(Tq, device="cuda") % n[d]].float()
        q = _unit(v + 0.1 * torch.randn(nq, Tq, DIM, generator=g, device="cuda"))
        return _grid(q).to(torch.bfloat16) if case["dtype"] == "bf16" else q


_built = {}  # corpora this process has indexed, the last used ones last


def _corpus(case):
    key = tuple(case[x] for x in _CORPUS_KEYS) + (case["call"] == "collab",)
    if key not in _built:
        c = _Corpus({x: case[x] for x in _CORPUS_KEYS})
        while _built and c.ntok + sum(o.ntok for o, _ in _built.values()) > KEEP_TOKENS:
            _built.pop(next(iter(_built)))[1][0].close()
        _built[key] = c, c.index(case["call"] == "collab")
    _built[key] = _built.pop(key)
    return _built[key]


def prepare(case, seed):
    corpus, built = _corpus(case)
    return dict(case=case, index=built[0], Q=corpus.queries(built, case, seed))


def run(state):
    c, idx, Q = state["case"], state["index"], state["Q"]
    if c["call"] == "collab":
        return idx.search_collab(Q, c["nprobe"], c["ncand"], c["kfb"], c["chunks"], c["k"], nthreads=16)
    if c["call"] == "rabitq":
        return idx.search_rabitq(Q, c["nprobe"], c["ncand"], c["k"])
    refine = chimera.REFINE_TOKEN if c["call"] == "refine" else chimera.REFINE_CENTROID
    return idx.search(Q, c["nprobe"], c["ncand"], c["k"], refine=refine)


def work(case):
    """Queries, centroids, probed posting entries and the candidates' codes read once, the results written once;
    the products of query tokens with centroids and with the candidates' tokens."""
    ntok, nq, Tq = case["ndocs"] * case["len_mean"], case["nq"], case["Tq"]
    scored = nq * min(case["ncand"], case["ndocs"]) * case["len_mean"]
    code = 20 if case["call"] == "rabitq" else 16 * case["nbits"] + 4
    probed = nq * Tq * case["nprobe"] * ntok / case["ncent"]
    if case["call"] == "refine":
        probed_bytes = min(ntok, probed) * (8 + 16 * case["nbits"])
    else:
        probed_bytes = min(ntok, probed) * 4
    bytes_ = (nq * Tq * DIM * (2 if case["dtype"] == "bf16" else 4) + case["ncent"] * DIM * 2 + probed_bytes
              + min(ntok, scored) * code + nq * case["k"] * 8)
    flops = 2.0 * DIM * Tq * (nq * case["ncent"] + scored)
    if case["call"] == "refine":
        flops += 2.0 * DIM * probed
    if case["call"] == "collab":
        flops += 2.0 * DIM * Tq * nq * case["kfb"] * case["len_mean"]
        bytes_ += min(ntok, nq * case["kfb"] * case["len_mean"]) * DIM * 2
    return dict(bytes=float(bytes_), flops=flops)


def tolerance(case):
    """Scores are exact multiples of 2^-22, rounded once (the RaBitQ ones: one rounding per token), and every list
    is ordered by (score, id): there is one right answer."""
    return "exact"


# ------------------------------------------------------------ the same in 64 bits
def _quantile(hist, num, den):
    n = int(hist.sum())
    return int(torch.searchsorted(torch.cumsum(hist, 0), min(num * n // den, n - 1), right=True)) - 4096


def _slices(beg, n):
    """Rows beg[i] .. beg[i] + n[i] - 1 for every i, and the i of each row."""
    i = torch.repeat_interleave(torch.arange(len(n), device=n.device), n)
    return beg[i] + torch.arange(len(i), device=n.device) - (torch.cumsum(n, 0) - n)[i], i


def _order(score, ids, most):
    """The `most` best by (score descending, id ascending): positions."""
    by_id = torch.argsort(ids)
    return by_id[torch.sort(score[by_id], descending=True, stable=True).indices[:most]]


def exact(case, seed):
    ntok = case["ndocs"] * case["len_mean"]
    if case["call"] == "rabitq" or ntok > 20_000_000:
        return None  # an encoder of its own, or a corpus that takes long to go through
    if case["nq"] * case["Tq"] * min(case["ncand"], case["ndocs"]) * case["len_mean"] > 6e9:
        return None
    corpus, built = _corpus(case)
    Q = _grid(corpus.queries(built, case, seed).float()).double()
    cent = corpus.cent.double()
    toks, cids = zip(*((tok, cid) for _, _, tok, cid in corpus.chunks()))
    tok, cid = torch.cat(toks), torch.cat(cids).long()
    # residual codes: buckets cut at the pooled quantiles, each read as its middle quantile
    B = 1 << case["nbits"]
    n0 = min(SAMPLE_TOKENS, len(toks[0]))
    res = torch.round((tok[:n0].float() - corpus.cent[cid[:n0]]) * 2048).int()
    hist = torch.bincount(res.flatten() + 4096, minlength=8193)
    cut = torch.tensor([_quantile(hist, i, B) for i in range(1, B)], device="cuda", dtype=torch.int32)
    wts = _grid(torch.tensor([_quantile(hist, 2 * u + 1, 2 * B) / 2048 for u in range(B)], device="cuda")).double()
    codes = torch.cat([torch.bucketize(torch.round((t.float() - corpus.cent[c.long()]) * 2048).int(), cut).byte()
                       for t, c in zip(toks, cids)])
    off = torch.from_numpy(corpus.off).cuda()
    doc_of = torch.repeat_interleave(torch.arange(case["ndocs"], device="cuda"), off[1:] - off[:-1])
    by_cent = torch.argsort(cid, stable=True)
    cent_n = torch.bincount(cid, minlength=case["ncent"])
    cent_off = torch.cumsum(cent_n, 0) - cent_n
    live = torch.ones(case["ndocs"], dtype=torch.bool, device="cuda")
    if corpus.deleted is not None:
        live[torch.from_numpy(corpus.deleted).cuda()] = False

    def doc_scores(docs, q, token_scores):
        rows, i = _slices(off[docs], off[docs + 1] - off[docs])
        best = torch.full((len(docs), len(q)), -math.inf, device="cuda", dtype=torch.float64)
        best.scatter_reduce_(0, i[:, None].expand(-1, len(q)), token_scores(rows), "amax")
        return best.sum(1)

    ids = torch.full((case["nq"], case["k"]), -1, device="cuda", dtype=torch.int64)
    out = torch.full((case["nq"], case["k"]), -math.inf, device="cuda", dtype=torch.float64)
    n_full = np.zeros(case["nq"], np.int64)
    ncand = min(case["ncand"], case["ndocs"])
    for qi, q in enumerate(Q):
        S = q @ cent.T
        top = torch.sort(S, dim=1, descending=True, stable=True).indices[:, :case["nprobe"]]
        rows, i = _slices(cent_off[top].flatten(), cent_n[top].flatten())
        t, j = by_cent[rows], i // case["nprobe"]
        s = S[j, top.flatten()[i]]
        if case["call"] == "refine":
            s = s + (wts[codes[t].long()] * q[j]).sum(1)
        part = torch.full((case["Tq"] * case["ndocs"],), -math.inf, device="cuda", dtype=torch.float64)
        part.scatter_reduce_(0, j * case["ndocs"] + doc_of[t], s, "amax")
        part = part.view(case["Tq"], case["ndocs"])
        hit = torch.isfinite(part)
        member = torch.nonzero(hit.any(0) & live).flatten()
        first = torch.where(hit, part, 0.0).sum(0)[member]
        cand = torch.sort(member[_order(first, member, ncand)]).values
        F = doc_scores(cand, q, lambda r: wts[codes[r].long()] @ q.T + S.T[cid[r]])
        if case["call"] == "collab":
            scored = {}
            for step in range(case["chunks"]):
                seen = min(len(cand), (step + 1) * ncand // case["chunks"])
                quota = -(-(step + 1) * case["kfb"] // case["chunks"])
                for p in _order(F[:seen], cand[:seen], quota).tolist():
                    scored.setdefault(p, None)
            at = torch.tensor(sorted(scored), device="cuda")
            cand = cand[at]
            F = doc_scores(cand, q, lambda r: tok[r].double() @ q.T)
            n_full[qi] = len(cand)
        best = _order(F, cand, case["k"])
        ids[qi, :len(best)], out[qi, :len(best)] = cand[best], F[best]
    return (ids, out, torch.from_numpy(n_full)) if case["call"] == "collab" else (ids, out)
