"""Document scoring by document (k_score_docs.hip) against the oracle, ids and
scores bit-exact, where it can go wrong: documents of one token, whole tiles
of 32 and one more, more tiles than the kernel keeps at once, odd and many
visits, both code widths, one and two blocks of query tokens.  300 queries
keep 250 or more of 300 documents, so each document has far more visits than
the rule asks for."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2608_23553_amd import build_index
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
