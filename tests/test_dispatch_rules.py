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


@pytest.mark.parametrize("chains,Tq,nprobe,ncent,M", [
    # measured faster through chains and the table (time against rank by rank)
    (True, 4, 8, 65_536, 1), (True, 16, 16, 65_536, 1), (True, 32, 16, 65_536, 1),    # 0.86, 0.84, 0.93
    (True, 32, 32, 65_536, 8), (True, 16, 4, 65_536, 8), (True, 32, 8, 262_144, 9),   # 0.80, 0.87, 0.94
    (True, 8, 32, 16_384, 1), (True, 16, 64, 65_536, 1),                              # 0.47, 0.44
    # measured slower
    (False, 32, 8, 65_536, 1), (False, 32, 4, 262_144, 1), (False, 32, 4, 65_536, 8),  # 1.11 to 1.22, 1.34, 1.03
    (False, 16, 4, 65_536, 1), (False, 4, 1, 65_536, 1), (False, 8, 1, 16_384, 1),     # 1.07 to 1.11, 1.09, 1.10
    (False, 32, 64, 65_536, 1), (False, 32, 32, 16_384, 1),                            # 1.13, 1.05
    (False, 64, 8, 65_536, 1), (False, 64, 32, 65_536, 1), (False, 64, 16, 262_144, 5),  # 1.02, 1.04, 1.03
])
def test_walk_through_chains_where_it_was_measured_faster(chains, Tq, nprobe, ncent, M):
    """Indexes of 64 dense lists, workgroups of M ranges."""
    f = _fn("_ZN7chimera14walk_by_chainsEiiiiii", ctypes.c_bool, *[ctypes.c_int] * 6)
    assert f(Tq, 32 if Tq <= 32 else 64, nprobe, ncent, 64, M) == chains
