"""Rules on sizes that choose between two ways of one step, asked on the CPU
through the library's own functions (C++ symbols of libchimera.so)."""
import ctypes

import pytest

from paper_2608_23553_amd import chimera


def _fn(symbol, restype, *argtypes):
    f = getattr(chimera.lib(), symbol)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


I32, I64 = ctypes.c_int32, ctypes.c_int64


def _split_select_bytes(nq, ndocs, ncand):
    """Scratch of the select split over chunks, from its arrays."""
    P = max(1, min(-(-16384 // nq), -(-ndocs // 4096)))
    per = (-(-ndocs // P) + 15) // 16 * 16
    cap = min(per, 4 * (ncand // P) + 1024)
    return nq * (32 + 4352 * 4 + P * (24 + 1024 + 8 + cap * 8)) + nq * P * (4 + cap * 8) + 1024


@pytest.mark.parametrize("nq", [1, 2, 7, 64, 127, 128, 1000])
def test_select_scratch_does_not_depend_on_the_select(nq):
    """What fits a scratch budget is the same whichever select runs."""
    f = _fn("_ZN7chimera20select_scratch_bytesElli", ctypes.c_size_t, I64, I64, I32)
    for ndocs in (1, 10, 4095, 4096, 4097, 8192, 24_576, 100_000, 1_000_000, 8_841_823, 12_582_912):
        for ncand in (1, 16, 1024, 4096, 100_000, 1 << 20):
            ncand = min(ncand, ndocs)
            assert f(nq, ndocs, ncand) == _split_select_bytes(nq, ndocs, ncand), (nq, ndocs, ncand)


# the corpora that both walks were timed on: documents, centroids, distinct centroids of a document's tokens
Z100 = (100_000, 16_384, 45)
Z1M = (1_000_000, 65_536, 49)
Z22 = (2_200_000, 262_144, 53)


@pytest.mark.parametrize("chains,Tq,nprobe,on,M", [
    # measured faster through chains and the table (time against rank by rank)
    (True, 4, 8, Z1M, 1), (True, 16, 16, Z1M, 1), (True, 32, 16, Z1M, 1),    # 0.86, 0.84, 0.93
    (True, 32, 32, Z1M, 8), (True, 16, 4, Z1M, 8), (True, 32, 8, Z22, 9),    # 0.80, 0.87, 0.94
    (True, 8, 32, Z100, 1), (True, 16, 64, Z1M, 1), (True, 32, 64, Z22, 3),  # 0.47, 0.44, 0.67
    (True, 13, 12, (4676, 4904, 31), 1),                                     # 0.44
    # measured slower
    (False, 32, 8, Z1M, 1), (False, 32, 4, Z22, 1), (False, 32, 4, Z1M, 8),  # 1.11 to 1.22, 1.34, 1.03
    (False, 16, 4, Z1M, 1), (False, 4, 1, Z1M, 1), (False, 8, 1, Z100, 1),   # 1.07 to 1.11, 1.09, 1.10
    (False, 32, 64, Z1M, 1), (False, 32, 32, Z100, 1),                       # 1.13, 1.05
    (False, 26, 22, (313_900, 15_644, 37), 1),                               # 1.17
    (False, 64, 8, Z1M, 1), (False, 64, 32, Z1M, 1), (False, 64, 16, Z22, 5),  # 1.02, 1.04, 1.03
])
def test_walk_through_chains_where_it_was_measured_faster(chains, Tq, nprobe, on, M):
    """Indexes of 64 dense lists, workgroups of M ranges."""
    ndocs, ncent, distinct = on
    f = _fn("_ZN7chimera14walk_by_chainsEiiilliii", ctypes.c_bool, I32, I32, I32, I64, I64, I32, I32, I32)
    assert f(Tq, 32 if Tq <= 32 else 64, nprobe, ndocs, ndocs * distinct, ncent, 64, M) == chains


_GROUPED = "_ZN7chimera17doc_score_groupedEliiillliiiib"


def _grouped(nq, Tq, nprobe, ncand, ndocs, L, ncent, *, longest=180, ndense=0, nbits=2, rq=False):
    f = _fn(_GROUPED, ctypes.c_bool, I64, I32, I32, I32, I64, I64, I64, I32, I32, I32, I32, ctypes.c_bool)
    ntok = int(ndocs * L)
    return f(nq, Tq, nprobe, ncand, ndocs, ntok, ntok, longest, ncent, ndense, nbits, rq)


# the corpora that both ways of scoring were timed on: documents, tokens a document, centroids
EVEN = dict(ndocs=100_000, L=64, ncent=16_384)
ZIPF = dict(ndocs=100_000, L=64, ncent=16_384, ndense=64)
M1 = dict(ndocs=1_000_000, L=70, ncent=65_536, ndense=64)
SHARD = dict(ndocs=2_200_000, L=70, ncent=262_144, ndense=64)
LONG = dict(ndocs=250_000, L=320, ncent=65_536, longest=512, nbits=4)


@pytest.mark.parametrize("by_doc,nq,Tq,nprobe,ncand,on", [
    # measured faster by document (its time against by query)
    (True, 256, 32, 4, 4096, EVEN), (True, 1024, 64, 4, 1024, EVEN), (True, 256, 4, 4, 8192, EVEN),  # 0.83 0.76 0.79
    (True, 256, 32, 4, 2048, ZIPF), (True, 1024, 16, 4, 1024, ZIPF),                                 # 0.94 0.80
    (True, 1024, 32, 4, 8192, M1), (True, 512, 32, 4, 4096, M1), (True, 1024, 4, 4, 8192, M1),       # 0.73 0.87 0.81
    (True, 1024, 32, 8, 16_384, SHARD), (True, 512, 8, 8, 16_384, SHARD),                            # 0.68 0.87
    (True, 128, 64, 8, 8192, LONG), (True, 32, 8, 8, 32_768, LONG),                                  # 0.50 0.72
    (True, 256, 32, 4, 16_384, dict(EVEN, longest=1200)),                                            # 0.77
    # measured slower
    (False, 64, 4, 4, 32_768, EVEN), (False, 64, 8, 4, 32_768, EVEN), (False, 16, 16, 4, 32_768, EVEN),  # 1.37 1.09 1.62
    (False, 64, 4, 4, 4096, ZIPF), (False, 64, 16, 4, 4096, ZIPF), (False, 64, 32, 4, 4096, ZIPF),   # 1.59 1.31 1.20
    (False, 256, 4, 4, 2048, ZIPF),                                                                  # 1.11
    (False, 256, 4, 4, 8192, M1), (False, 256, 16, 4, 8192, M1), (False, 512, 4, 4, 4096, M1),       # 1.38 1.11 1.23
    (False, 256, 8, 8, 16_384, SHARD), (False, 4, 64, 8, 32_768, LONG),                              # 1.15 1.24
    (False, 938, 51, 5, 87, dict(ndocs=2211, L=77, ncent=2685, ndense=64, nbits=4)),                 # 1.73
    (False, 938, 51, 5, 400, dict(ndocs=2211, L=77, ncent=2685, ndense=64, nbits=4)),                # 1.31
    (False, 300, 51, 5, 400, dict(ndocs=2211, L=77, ncent=2685, ndense=64, nbits=4)),                # 1.27
    (False, 762, 32, 20, 278, dict(ndocs=4309, L=77, ncent=1714, ndense=64)),                        # 1.06
    # one document keeps the chip waiting
    (False, 256, 32, 4, 4096, dict(EVEN, longest=1200)), (False, 1024, 32, 4, 4096, dict(EVEN, longest=40_000)),
    (False, 256, 32, 8, 8192, dict(M1, longest=2000)), (False, 256, 32, 4, 4096, dict(EVEN, L=74.7, longest=600)),
])
def test_scoring_by_document_where_it_was_measured_faster(by_doc, nq, Tq, nprobe, ncand, on):
    assert _grouped(nq, Tq, nprobe, ncand, **on) == by_doc


@pytest.mark.parametrize("by_doc,nq,Tq,ncand,on", [
    (True, 256, 32, 4096, EVEN), (True, 128, 32, 8192, ZIPF), (True, 512, 64, 512, dict(EVEN, ndocs=20_000)),
    (True, 256, 32, 16_384, dict(EVEN, longest=2400)), (True, 256, 64, 4096, dict(EVEN, longest=600)),
    (False, 512, 32, 512, dict(EVEN, ndocs=20_000)), (False, 512, 32, 512, ZIPF),  # 1.07 1.04
    (False, 256, 64, 4096, dict(EVEN, longest=2400)), (False, 256, 32, 4096, dict(EVEN, longest=2400)),  # 1.41 1.72
])
def test_rabitq_scoring_by_document_where_it_was_measured_faster(by_doc, nq, Tq, ncand, on):
    assert _grouped(nq, Tq, 4, ncand, **on, rq=True) == by_doc
