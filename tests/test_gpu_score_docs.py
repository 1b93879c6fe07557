"""Document scoring by document (k_score_docs.hip) against the oracle, ids and
scores bit-exact, where it can go wrong: documents of one token, whole tiles
of 32 and one more, more tiles than the kernel keeps at once, odd and many
visits, both code widths, one and two blocks of query tokens.  The first tests'
300 queries keep 250 or more of 300 documents; where their batches are too
small for the library's rule, the later ones ask it and are larger."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2608_23553_amd import Builder, build_index, chimera
from synth import k_to_bf16_bits
from util_corpus import rand_grid
from util_build import product_builder
from util_gpu import check_search, q_tensor, say, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits", [2, 4])
@pytest.mark.parametrize("Tq,lo,hi", [(5, 1, 80), (32, 31, 65), (32, 150, 420), (33, 1, 80), (64, 120, 420)])
def test_by_document(nbits, Tq, lo, hi):
    w, c, k, cl, oi, idx = setup("tiny", ndocs=300, ncent=64, nbits=nbits, len_kind=2, len_lo=lo, len_hi=hi)
    q, _ = c.queries(300, Tq, query_seed=Tq + hi)
    check_search(idx, oi, q, 16, 299 if Tq == 33 else 300, 40, "bf16", f"by document, Tq={Tq}, {lo}..{hi} tokens")


def test_tokens_past_fp16_are_scored_by_query():
    """A centroid on an axis: its component 1 plus a residual is no fp16 value
    in general, so this index keeps to the scoring by query."""
    rng = np.random.default_rng(11)
    cent = rand_grid(rng, (64, 128))
    cent[0] = 0
    cent[0, 3] = 2048
    lens = rng.integers(1, 90, 300).astype(np.int32)
    cid = rng.integers(0, 64, int(lens.sum())).astype(np.int32)
    cid[::5] = 0
    v = cent[cid] / 2048 + 0.05 * rng.standard_normal((len(cid), 128))
    tok = oracle.grid_f32((v / np.linalg.norm(v, axis=1, keepdims=True)).astype(np.float32))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    oi = oracle.OracleIndex(cent, off, cid, 2, tok_k=tok)
    idx = build_index(k_to_bf16_bits(cent), 2, lambda: [(k_to_bf16_bits(tok), cid, lens)]).upload(0)
    q = rand_grid(rng, (300, 32, 128))
    q[:, 0] = cent[0]
    say("axis centroid")
    check_search(idx, oi, q, 16, 300, 40, "bf16", "axis centroid")
    torch.cuda.synchronize()


@pytest.mark.parametrize("Tq,lo,hi", [(5, 1, 80), (32, 31, 65), (32, 150, 300), (64, 120, 260)])
def test_rabitq_by_document(Tq, lo, hi):
    """The RaBitQ 1-bit scores of the same kind of batch; sampled queries."""
    w, c, k, cl, oi, _ = setup("tiny", ndocs=300, ncent=64, len_kind=2, len_lo=lo, len_hi=hi)
    signs = synth.rotation_signs(29)
    idx = product_builder(c, w.nbits, rabitq_signs=signs).upload(0)
    codes, _, g1 = oracle.rabitq_encode(k, signs, 4)
    q, _ = c.queries(300, Tq, query_seed=Tq + hi)
    q[3] = 0
    say("rabitq by document", Tq, lo, hi)
    ids, scores = idx.search_rabitq(q_tensor(q, "bf16"), 16, 300, 40)
    torch.cuda.synchronize()
    for i in (0, 3, 150, 299):
        ref = oracle.search_rabitq(oi, q[i:i + 1], 16, 300, 40, signs, 4, codes, g1)
        assert np.array_equal(ids[i].cpu().numpy(), ref["ids"][0]), i
        assert np.array_equal(scores[i].cpu().numpy(), ref["scores"][0]), i
    idx.close()


def _goes_by_document(idx, nq, Tq, nprobe, ncand, nbits=2, rq=False):
    """The library's rule, for these corpora of 64 centroids (every list is dense)."""
    f = chimera.lib()._ZN7chimera17doc_score_groupedEliiillliiiib
    i32, i64 = ctypes.c_int32, ctypes.c_int64
    f.restype, f.argtypes = ctypes.c_bool, [i64, i32, i32, i32, i64, i64, i64, i32, i32, i32, i32, ctypes.c_bool]
    i = idx.info()
    return f(nq, Tq, nprobe, ncand, i["ndocs"], i["ntokens"], i["nnz"], i["max_doc_len"], i["ncent"], 64, nbits, rq)


def _np(out):
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


def _by_query(search, Q, nprobe, ncand, k, step):
    """The same searches in batches too small to go by document."""
    parts = [_np(search(Q[i:i + step], nprobe, ncand, k)) for i in range(0, len(Q), step)]
    return [np.concatenate(x) for x in zip(*parts)]


@pytest.mark.parametrize("nbits", [2, 4])
@pytest.mark.parametrize("Tq,lo,hi", [(5, 1, 80), (32, 31, 65), (32, 150, 420), (33, 1, 80), (64, 120, 420)])
def test_by_document_is_by_query(nbits, Tq, lo, hi):
    """200 queries of 2,999 candidates at once and 20 at a time, bit for bit,
    and sampled ones against the oracle."""
    w, c, k, cl, oi, idx = setup("tiny", ndocs=3000, ncent=64, nbits=nbits, len_kind=2, len_lo=lo, len_hi=hi)
    assert _goes_by_document(idx, 200, Tq, 16, 2999, nbits) and not _goes_by_document(idx, 20, Tq, 16, 2999, nbits)
    q, _ = c.queries(200, Tq, query_seed=Tq + lo)
    Q = q_tensor(q, "bf16")
    say("by document and by query", nbits, Tq, lo, hi)
    ids, scores = _np(idx.search(Q, 16, 2999, 40))
    ids2, scores2 = _by_query(idx.search, Q, 16, 2999, 40, 20)
    assert np.array_equal(ids, ids2) and np.array_equal(scores, scores2)
    sample = [0, 7, 199]
    ref = oi.search(q[sample], 16, 2999, 40)
    assert np.array_equal(ids[sample], ref["ids"]) and np.array_equal(scores[sample], ref["scores"])


@pytest.mark.parametrize("Tq,lo,hi", [(5, 1, 80), (32, 31, 65), (32, 150, 300), (64, 120, 260)])
def test_rabitq_by_document_is_by_query(Tq, lo, hi):
    """(The scoring by query is compared with the oracle above.)"""
    w, c, _, _, _, _ = setup("tiny", ndocs=1100, ncent=64, len_kind=2, len_lo=lo, len_hi=hi)
    idx = product_builder(c, w.nbits, rabitq_signs=synth.rotation_signs(31)).upload(0)
    assert _goes_by_document(idx, 90, Tq, 16, 1099, rq=True) and not _goes_by_document(idx, 45, Tq, 16, 1099, rq=True)
    q, _ = c.queries(90, Tq, query_seed=Tq + lo)
    q[3] = 0
    Q = q_tensor(q, "bf16")
    say("rabitq by document and by query", Tq, lo, hi)
    ids, scores = _np(idx.search_rabitq(Q, 16, 1099, 40))
    ids2, scores2 = _by_query(idx.search_rabitq, Q, 16, 1099, 40, 45)
    assert np.array_equal(ids, ids2) and np.array_equal(scores, scores2)
    idx.close()


def _fresh(monkeypatch, c, nbits, **kw):
    """An index of its own (no arena yet) that counts its sub-batches."""
    monkeypatch.setenv("CHIMERA_STAGE_TIMING", "1")
    return product_builder(c, nbits, **kw).upload(0)


def _passes(idx, nq):
    """Queries of a sub-batch of the last search, and its number of sub-batches."""
    n = int(idx.stage_times()[6])
    return -(-nq // n), n


def test_sub_batches_by_document(monkeypatch):
    """Several sub-batches that go by document, the last one shorter, residual
    and RaBitQ; the same as in one pass."""
    w, c, _, _, _, one = setup("tiny", ndocs=1100, ncent=64, len_kind=2, len_lo=31, len_hi=65)
    signs = synth.rotation_signs(31)
    idx = _fresh(monkeypatch, c, w.nbits, rabitq_signs=signs)
    q, _ = c.queries(391, 32, query_seed=77)
    Q = q_tensor(q, "bf16")
    want = _np(one.search(Q, 16, 1099, 40))
    want_rq = _np(idx.search_rabitq(Q, 16, 1099, 40))
    assert _passes(idx, 391) == (391, 1)
    monkeypatch.setenv("CHIMERA_SCRATCH_MB", "16")
    for rq, search, ref in ((False, idx.search, want), (True, idx.search_rabitq, want_rq)):
        say("sub-batches by document", rq)
        got = _np(search(Q, 16, 1099, 40))
        B, n = _passes(idx, 391)
        say(n, "sub-batches of", B)
        assert n > 1 and 391 % B and _goes_by_document(idx, B, 32, 16, 1099, rq=rq)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    idx.close()


def test_arena_that_does_not_fit_by_document(monkeypatch):
    """Sub-batches halved because the device refuses the arena: once with the
    halves still by document, and down to where they go by query (whose S^T
    then enters the scratch)."""
    w, c, _, _, _, one = setup("tiny", ndocs=1100, ncent=64, len_kind=2, len_lo=31, len_hi=65)
    q, _ = c.queries(700, 32, query_seed=78)
    Q = q_tensor(q, "bf16")
    want = _np(one.search(Q, 16, 1099, 40))
    routes = {}
    for mb in (48, 24, 12, 6):
        idx = _fresh(monkeypatch, c, w.nbits)
        monkeypatch.setenv("CHIMERA_SCRATCH_DEVICE_MB", str(mb))
        got = _np(idx.search(Q, 16, 1099, 40))
        monkeypatch.delenv("CHIMERA_SCRATCH_DEVICE_MB")
        B, n = _passes(idx, 700)
        routes[n, _goes_by_document(idx, B, 32, 16, 1099)] = mb
        say(mb, "MB:", n, "sub-batches of", B)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        idx.close()
    assert any(n > 1 and docs for n, docs in routes) and any(not docs for _, docs in routes), routes


def test_one_query_that_fits_by_query_only(monkeypatch):
    """One query that keeps all of 66,000 documents of 480 tokens goes by
    document, which needs two words a document more than the centroid scores of
    64 centroids: where the device has only the latter, it is answered by query."""
    monkeypatch.setenv("CHIMERA_STAGE_TIMING", "1")
    rng = np.random.default_rng(12)
    cent = rand_grid(rng, (64, 128))
    cid = rng.integers(0, 64, 100 * 480).astype(np.int32)
    v = cent[cid] / 2048 + 0.05 * rng.standard_normal((len(cid), 128))
    tok = k_to_bf16_bits(oracle.grid_f32((v / np.linalg.norm(v, axis=1, keepdims=True)).astype(np.float32)))
    b = Builder(k_to_bf16_bits(cent), 2)
    b.add_residuals(tok, cid)
    b.freeze()
    for _ in range(660):  # a hundred documents, over and over
        b.add_docs(tok, cid, np.full(100, 480, np.int32))
    idx = b.upload(0)
    b.close()
    assert _goes_by_document(idx, 1, 64, 32, 66_000)
    Q = q_tensor(rand_grid(rng, (1, 64, 128)), "bf16")
    monkeypatch.setenv("CHIMERA_SCRATCH_DEVICE_MB", "3")
    say("one query, 3 MB")
    got = _np(idx.search(Q, 32, 66_000, 40))
    monkeypatch.delenv("CHIMERA_SCRATCH_DEVICE_MB")
    want = _np(idx.search(Q, 32, 66_000, 40))
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    idx.close()


def test_by_document_with_deletions_and_without_allocation():
    w, c, _, _, oi, _ = setup("tiny", ndocs=1100, ncent=64, len_kind=2, len_lo=31, len_hi=65)
    idx = product_builder(c, w.nbits).upload(0)
    gone = np.zeros(1100, bool)
    gone[np.random.default_rng(9).choice(1100, 150, replace=False)] = True
    idx.delete(np.nonzero(gone)[0])
    assert _goes_by_document(idx, 400, 32, 16, 1099)
    q, _ = c.queries(400, 32, query_seed=79)
    Q = q_tensor(q, "bf16")
    for label in ("bitmap", "compacted"):
        say("by document,", label)
        ids, scores = _np(idx.search(Q, 16, 1099, 40))
        na = torch.full((400, 40), -7, dtype=torch.int32, device="cuda"), torch.zeros((400, 40), device="cuda")
        rc = chimera.lib().chimera_search_noalloc(idx._h, Q.data_ptr(), chimera.BF16, 400, 32, 128, 16, 1099, 40,
                                                  na[0].data_ptr(), na[1].data_ptr(),
                                                  torch.cuda.current_stream().cuda_stream)
        assert rc == chimera.OK, chimera.last_error()
        na = _np(na)
        assert np.array_equal(ids, na[0]) and np.array_equal(scores, na[1])
        sample = [0, 199, 399]
        ref = oracle.search_deleted(oi, q[sample], 16, 1099, 40, gone)
        assert np.array_equal(ids[sample], ref["ids"])
        idx.compact()
    idx.close()


def test_an_index_of_zeros_takes_any_query():
    """Centroids and weights of 0 bound no query's norm, so its components may
    be past fp16: every score is 0, in a batch as for one query."""
    lens = np.full(1100, 48, np.int32)
    tok = np.zeros((1100 * 48, 128), np.uint16)
    cid = (np.arange(len(tok)) % 64).astype(np.int32)
    idx = build_index(np.zeros((64, 128), np.uint16), 2, lambda: [(tok, cid, lens)]).upload(0)
    assert idx.info()["q_norm_limit"] > 1e8 and _goes_by_document(idx, 400, 31, 16, 1099)
    Q = torch.full((400, 31, 128), 1e6, device="cuda")
    say("zeros")
    one = _np(idx.search(Q[:1], 16, 1099, 40))
    ids, scores = _np(idx.search(Q, 16, 1099, 40))
    assert (one[1] == 0).all() and (scores == 0).all()
    assert (ids == one[0]).all()
    idx.close()
