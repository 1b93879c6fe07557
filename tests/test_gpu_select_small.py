"""The small batch's select (k_keep_list, k_keep_cut) and the top-k against the
oracle, at the edges of their chunks (4096 documents), of the lists and of the
registers: no more hits than candidates, one candidate, whole documents sets
tied (the query's list overflows and F' is read instead), more entries than a
thread keeps, and k of 1 up to every candidate."""
import numpy as np
import pytest
import torch

from util_build import product_builder
from util_gpu import check_search, q_tensor, say, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndocs", [4095, 4096, 4097, 12_289])
@pytest.mark.parametrize("ncand,k", [(1, 1), (37, 37), (4096, 100)])
def test_chunk_edges(ndocs, ncand, k):
    w, c, _, _, oi, idx = setup("tiny", ndocs=ndocs, ncent=256, len_kind=2, len_lo=1, len_hi=4)
    q, _ = c.queries(3, 32, query_seed=ndocs + ncand)
    cand, keys, nval = idx.prune(q_tensor(q, "bf16"), 4, ncand)
    torch.cuda.synchronize()
    ref = oi.prune(q, 4, min(ncand, ndocs))
    for i in range(3):
        n = ref["n_cand"][i]
        order = np.argsort(ref["cand"][i, :n])
        assert nval[i].item() == n
        assert np.array_equal(cand[i, :n].cpu().numpy(), ref["cand"][i, :n][order])
        assert np.array_equal(keys[i, :n].cpu().numpy(), ref["cand_keys"][i, :n][order])
        assert (cand[i, n:] == -1).all()
    check_search(idx, oi, q, 4, ncand, k, "bf16", f"{ndocs} documents, ncand {ncand}, k {k}")


@pytest.mark.parametrize("ncand,k", [(10, 3), (20_000, 1), (20_000, 5000), (30_000, 8192)])
def test_ties_and_long_lists(ncand, k):
    """30,000 documents over 64 centroids: an all-zero query ties every hit at
    F' = 0 and every score at 0, more than a list of 4 ncand + 4096 holds for
    ncand = 10; with ncand = 20,000 the list (and the top-k's input) is longer
    than the registers take."""
    w, c, _, _, oi, idx = setup("tiny", ndocs=30_000, ncent=64, len_kind=2, len_lo=1, len_hi=3)
    q, _ = c.queries(3, 8, query_seed=5)
    q[1] = 0
    say("ties", ncand, k)
    check_search(idx, oi, q, 32, ncand, k, "bf16", f"ties, ncand {ncand}, k {k}")


def _check_prune(idx, oi, q, nprobe, ncand):
    say("prune", q.shape, nprobe, ncand)
    cand, keys, nval = (x.cpu().numpy() for x in idx.prune(q_tensor(q, "bf16"), nprobe, ncand))
    ref = oi.prune(q, nprobe, ncand)
    for i in range(len(q)):
        n = ref["n_cand"][i]
        order = np.argsort(ref["cand"][i, :n])
        assert nval[i] == n, i
        assert np.array_equal(cand[i, :n], ref["cand"][i, :n][order]), i
        assert np.array_equal(keys[i, :n], ref["cand_keys"][i, :n][order]), i
        assert (cand[i, n:] == -1).all() and (keys[i, n:] == 0).all(), i


@pytest.mark.parametrize("ndocs,ncand", [
    (200_001, 10),       # lists past their capacity: the passes read F'
    (200_001, 30_000),   # lists longer than the registers, within their capacity
    (200_001, 199_000),  # every hit kept, from its chunk's count
    (4096, 1),           # one chunk whose list is past its capacity
])
def test_lists_cut_by_many_workgroups(ndocs, ncand):
    """A tied query, a query of four tokens (few bins of the first pass, so
    most documents are in the one that is cut) and two of 32, in one batch."""
    w, c, _, _, oi, idx = setup("tiny", ndocs=ndocs, ncent=64, len_kind=2, len_lo=1, len_hi=3)
    q, _ = c.queries(4, 32, query_seed=ncand)
    q[1] = 0
    q[2, 4:] = 0
    _check_prune(idx, oi, q, 32, ncand)


def test_a_long_list_is_not_cut_by_one_workgroup(monkeypatch):
    """One query whose million documents all tie: the select's three passes
    over F' are spread over the chip, well under the 1,600 us that one
    workgroup takes over them."""
    monkeypatch.setenv("CHIMERA_STAGE_TIMING", "1")
    w, c, _, _, _, _ = setup("tiny", ndocs=1_000_000, ncent=64, len_kind=2, len_lo=1, len_hi=2)
    idx = product_builder(c, w.nbits).upload(0)
    q = torch.zeros((1, 32, 128), device="cuda")
    best = {}
    for ncand in (64, 30_000, 500_000):
        for _ in range(8):
            idx.search(q, 32, ncand, 10)
            best[ncand] = min(best.get(ncand, 1e9), 1e3 * float(idx.stage_times()[3]))
    say("select of one query, us:", best)
    assert max(best.values()) < 300, best
    idx.close()


@pytest.mark.parametrize("ncand", [1024, 1025, 4096, 4097])
def test_topk_at_the_edges_of_its_registers(ncand):
    """1, 4 and 16 keys a thread; k of 1, some and every candidate; a tied query."""
    w, c, _, _, oi, idx = setup("tiny", ndocs=12_289, ncent=256, len_kind=2, len_lo=1, len_hi=4)
    q, _ = c.queries(3, 32, query_seed=ncand)
    q[1] = 0
    for k in (1, 37, ncand):
        check_search(idx, oi, q, 32, ncand, k, "bf16", f"top-k, ncand {ncand}, k {k}")


def test_topk_of_few_candidates_keeps_two_workgroups_a_cu(monkeypatch):
    """512 queries of 64 candidates take little longer in the top-k than 256
    (1.3 times; 1.6 when a CU holds one workgroup)."""
    monkeypatch.setenv("CHIMERA_STAGE_TIMING", "1")
    w, c, _, _, _, _ = setup("tiny", ndocs=12_289, ncent=256, len_kind=2, len_lo=1, len_hi=4)
    idx = product_builder(c, w.nbits).upload(0)
    Q = q_tensor(c.queries(512, 8, query_seed=1)[0], "bf16")
    best = {}
    for _ in range(40):
        for nq in (256, 512):
            idx.search(Q[:nq], 4, 64, 10)
            best[nq] = min(best.get(nq, 1e9), 1e3 * float(idx.stage_times()[5]))
    say("top-k, us:", best)
    assert best[512] < 1.45 * best[256], best
    idx.close()
