"""The candidate walk of an index with dense lists against the oracle: ranges
through chains of entries and the dense groups' table, ranges with more
entries than the chains hold (walked rank by rank), queries with more dense
groups than the table takes, documents with more entries than a lane sorts,
query tokens that share centroids, both token-mask widths and deletions."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2608_23553_amd import chimera
from util_gpu import check_search, q_tensor, say, setup

pytestmark = pytest.mark.gpu


def _check_prune(idx, ref, q, nprobe, ncand, label):
    say("prune", label)
    cand, keys, nval = (x.cpu().numpy() for x in idx.prune(q_tensor(q, "bf16"), nprobe, ncand))
    for i in range(len(q)):
        n = ref["n_cand"][i]
        order = np.argsort(ref["cand"][i, :n])
        assert nval[i] == n, (label, i)
        assert np.array_equal(cand[i, :n], ref["cand"][i, :n][order]), (label, i)
        assert np.array_equal(keys[i, :n], ref["cand_keys"][i, :n][order]), (label, i)


@pytest.mark.parametrize("ndocs,ncent,nprobe,Tq", [
    (4096, 16_384, 12, 32),  # few entries, one whole range
    (9001, 8192, 16, 32),    # 512 lists, a ragged last range
    (9001, 8192, 40, 32),    # windows of two entries, many dense groups
    (12_289, 600, 9, 32),    # more entries in a range than the chains hold
    (5000, 4096, 12, 64),    # 64-bit masks, ranges of 2048
    (6145, 700, 30, 64),     # 64-bit masks and a full walk rank by rank
    (4097, 2048, 1, 5),      # one rank, few tokens
    (9001, 8192, 4, 32),     # few ranks
])
def test_prune(ndocs, ncent, nprobe, Tq):
    w, c, _, cl, oi, idx = setup("1m", ndocs=ndocs, ncent=ncent)
    q, _ = c.queries(5, Tq, query_seed=ncent + nprobe)
    q[4] = np.repeat(q[4, :(Tq + 3) // 4], 4, axis=0)[:Tq]  # tokens four times over
    ncand = ndocs  # every hit with its F'
    _check_prune(idx, oi.prune(q, nprobe, ncand), q, nprobe, ncand, f"{ndocs} docs, {ncent} cents, np {nprobe}, Tq {Tq}")
    check_search(idx, oi, q, nprobe, 300, 20, "bf16", "search")


def test_group_counts_on_both_sides_of_the_table():
    """Queries of the cases above fall on both sides of the 11 groups that the
    table takes: with nprobe 1 to 40 their dense groups run from none to many."""
    w, c, _, cl, oi, idx = setup("1m", ndocs=9001, ncent=8192)
    docs = np.repeat(np.arange(9001), c.lengths)
    in_list = np.zeros(8192, np.int64)
    np.add.at(in_list, np.unique(np.stack([cl, docs]), axis=1)[0], 1)
    dense = set(np.argsort(-in_list, kind="stable")[:64]) & set(np.nonzero(in_list * 16 > 9001)[0])
    q, _ = c.queries(24, 32, query_seed=77)
    groups = []
    for qq in q:
        ids = np.asarray(oracle.probe(oracle.centroid_scores(qq, c.centroids_k), 16)[0])
        groups.append(sum(len(dense & set(ids[:, r])) for r in range(16)))
    assert min(groups) <= 11 < max(groups), groups
    _check_prune(idx, oi.prune(q, 16, 9001), q, 16, 9001, f"groups {min(groups)}..{max(groups)}")


def test_deleted_documents():
    w, c, _, _, oi, _ = setup("1m", ndocs=9001, ncent=8192)
    from util_build import product_builder
    idx = product_builder(c, w.nbits).upload(0)
    gone = np.random.default_rng(3).choice(9001, 1500, replace=False)
    idx.delete(gone)
    q, _ = c.queries(4, 32, query_seed=9)
    ids, _ = idx.search(q_tensor(q, "bf16"), 16, 400, 30)
    torch.cuda.synchronize()
    deleted = np.zeros(9001, bool)
    deleted[gone] = True
    ref = oracle.search_deleted(oi, q, 16, 400, 30, deleted)
    assert np.array_equal(ids.cpu().numpy(), ref["ids"])


@pytest.mark.parametrize("row,nprobe", [(42, 11), (70, 12)])
def test_chains_overflow_in_a_workgroups_second_range(row, nprobe):
    """A workgroup of two ranges whose second holds more entries than the
    chains: its histogram and its lists go on rank by rank.  17,000 queries
    make the walk's workgroups take two of the four ranges each."""
    w, c, _, cl, oi, idx = setup("1m", ndocs=16_384, ncent=16_384)
    q, _ = c.queries(120, 32, query_seed=5)
    pairs = np.unique(np.stack([cl, np.repeat(np.arange(16_384), c.lengths)]), axis=1)
    count = np.zeros((16_384, 4), np.int64)
    np.add.at(count, (pairs[0], pairs[1] // 4096), 1)
    total = count.sum(1)
    dense = np.nonzero((total * 16 > 16_384) & (np.argsort(np.argsort(-total, kind="stable")) < 64))[0]
    ids = np.asarray(oracle.probe(oracle.centroid_scores(q[row], c.centroids_k), nprobe)[0])
    ranks = [np.setdiff1d(ids[:, r], dense) for r in range(nprobe)]
    entries = sum(count[x].sum(0) for x in ranks)
    assert sum(len(np.intersect1d(ids[:, r], dense)) for r in range(nprobe)) <= 11
    assert any(entries[a] <= 4096 < entries[a + 1] for a in (0, 2)), entries
    few = q[[row, 0, 1, 2, 3]]
    say("prune 17,000 queries", row, nprobe)
    many = q_tensor(few, "bf16").repeat(3400, 1, 1)
    cand, keys, nval = idx.prune(many, nprobe, 500)
    cand, keys, nval = (x.view(3400, 5, *x.shape[1:]) for x in (cand, keys, nval))
    ref = oi.prune(few, nprobe, 500)
    for i in range(5):
        assert ref["n_cand"][i] == 500 and bool((nval[:, i] == 500).all())
        order = np.argsort(ref["cand"][i, :500])
        assert np.array_equal(cand[0, i].cpu().numpy(), ref["cand"][i, :500][order]), i
        assert np.array_equal(keys[0, i].cpu().numpy(), ref["cand_keys"][i, :500][order]), i
        assert bool((cand[:, i] == cand[0, i]).all()) and bool((keys[:, i] == keys[0, i]).all()), i


def _by_chains(idx, Tq, nprobe, ndense, M):
    f = chimera.lib()._ZN7chimera14walk_by_chainsEiiilliii
    i32, i64 = ctypes.c_int32, ctypes.c_int64
    f.restype, f.argtypes = ctypes.c_bool, [i32, i32, i32, i64, i64, i32, i32, i32]
    i = idx.info()
    return f(Tq, 32 if Tq <= 32 else 64, nprobe, i["ndocs"], i["nnz"], i["ncent"], ndense, M)


def _dense(c, cl, ndocs, ncent, R=4096):
    """Documents of each centroid's list in each range of R, and the dense lists."""
    pairs = np.unique(np.stack([cl, np.repeat(np.arange(ndocs), c.lengths)]), axis=1)
    count = np.zeros((ncent, -(-ndocs // R)), np.int64)
    np.add.at(count, (pairs[0], pairs[1] // R), 1)
    total = count.sum(1)
    return count, np.nonzero((total * 16 > ndocs) & (np.argsort(np.argsort(-total, kind="stable")) < 64))[0]


@pytest.mark.parametrize("ndocs,ncent,nprobe,Tq,lens", [
    (9001, 65_536, 16, 32, None),        # 10 to 15 dense groups: both ways in one batch; a ragged last range
    (9001, 65_536, 32, 32, None),        # two lists a thread
    (4096, 16_384, 16, 16, None),        # one whole range
    (9001, 8192, 16, 8, (50, 150)),      # long chains
    (16_384, 16_384, 16, 16, (50, 150)),  # some ranges hold more entries than the chains
    (5000, 4096, 9, 7, None),            # few tokens
])
def test_prune_by_chains(ndocs, ncent, nprobe, Tq, lens):
    kw = dict(len_kind=2, len_lo=lens[0], len_hi=lens[1]) if lens else {}
    w, c, _, cl, oi, idx = setup("1m", ndocs=ndocs, ncent=ncent, **kw)
    assert _by_chains(idx, Tq, nprobe, len(_dense(c, cl, ndocs, ncent)[1]), 1)
    q, _ = c.queries(24, Tq, query_seed=5)
    q[4] = np.repeat(q[4, :(Tq + 3) // 4], 4, axis=0)[:Tq]  # tokens four times over
    _check_prune(idx, oi.prune(q, nprobe, ndocs), q, nprobe, ndocs, f"chains: {ndocs} {ncent} {nprobe} {Tq} {lens}")


def test_second_range_past_the_chains_by_chains():
    """A workgroup of two ranges (17,000 queries make it so) whose second holds
    more entries than the chains: what follows is walked rank by rank."""
    ndocs = ncent = 16_384
    w, c, _, cl, oi, idx = setup("1m", ndocs=ndocs, ncent=ncent, len_kind=2, len_lo=50, len_hi=150)
    count, dense = _dense(c, cl, ndocs, ncent)
    assert _by_chains(idx, 16, 16, len(dense), 2)
    few = c.queries(400, 16, query_seed=5)[0][[14, 0, 1, 2, 3]]
    ids = np.asarray(oracle.probe(oracle.centroid_scores(few[0], c.centroids_k), 16)[0])
    entries = sum(count[np.setdiff1d(ids[:, r], dense)].sum(0) for r in range(16))
    assert sum(len(np.intersect1d(ids[:, r], dense)) for r in range(16)) <= 11
    assert any(entries[a] <= 4096 < entries[a + 1] for a in (0, 2)), entries
    say("prune 17,000 queries by chains")
    cand, keys, nval = idx.prune(q_tensor(few, "bf16").repeat(3400, 1, 1), 16, 500)
    cand, keys, nval = (x.view(3400, 5, *x.shape[1:]) for x in (cand, keys, nval))
    ref = oi.prune(few, 16, 500)
    for i in range(5):
        assert ref["n_cand"][i] == 500 and bool((nval[:, i] == 500).all())
        order = np.argsort(ref["cand"][i, :500])
        assert np.array_equal(cand[0, i].cpu().numpy(), ref["cand"][i, :500][order]), i
        assert np.array_equal(keys[0, i].cpu().numpy(), ref["cand_keys"][i, :500][order]), i
        assert bool((cand[:, i] == cand[0, i]).all()) and bool((keys[:, i] == keys[0, i]).all()), i


@pytest.mark.parametrize("nprobe,Tq", [(8, 64), (24, 64), (32, 64), (8, 32), (24, 32), (64, 32)])
def test_prune_rank_by_rank(nprobe, Tq):
    """Either mask width with one, two and four lists a thread."""
    w, c, _, cl, oi, idx = setup("1m", ndocs=9001, ncent=8192)
    assert not _by_chains(idx, Tq, nprobe, len(_dense(c, cl, 9001, 8192)[1]), 1)
    q, _ = c.queries(9, Tq, query_seed=nprobe)
    _check_prune(idx, oi.prune(q, nprobe, 9001), q, nprobe, 9001, f"ranks: {nprobe} {Tq}")
