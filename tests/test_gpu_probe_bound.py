"""The probe with a sampled row bound against the oracle: a ragged last tile of
centroids, a sample of an odd number of tiles, one and more probes per token,
an all-zero query (every centroid ties)."""
import numpy as np
import pytest
import torch

import oracle
from util_gpu import q_tensor, say, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncent,nprobe", [(8219, 1), (8219, 5), (8219, 9), (65_537, 16), (65_537, 40)])
def test_sampled_bound(ncent, nprobe):
    w, c, _, _, _, idx = setup("tiny", ndocs=64, ncent=ncent)
    q, _ = c.queries(130, 32, query_seed=nprobe)
    q[7] = 0
    say("probe", ncent, nprobe)
    ci, ck = idx.probe(q_tensor(q, "bf16"), nprobe)
    torch.cuda.synchronize()
    ci, ck = ci.cpu().numpy(), ck.cpu().numpy()
    for i in (0, 1, 7, 64, 129):
        ids, keys = oracle.probe(oracle.centroid_scores(q[i], c.centroids_k), nprobe)
        assert np.array_equal(ci[i], ids), i
        assert np.array_equal(ck[i].astype(np.int64), keys), i
