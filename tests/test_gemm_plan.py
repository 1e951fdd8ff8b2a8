"""The tile plans of the token passes' GEMMs (host arithmetic): every shape gets a launch its kernels
accept, and the workspace holds the partial sums of every pass it may run."""
import ctypes as C
import os

import pytest

BN = (256, 256, 128, 128, 128, 128, 64, 256)


@pytest.fixture(scope="module")
def probe():
    from paper_2508_10259_amd.build import PROBE_LIB
    if not os.path.exists(PROBE_LIB):
        pytest.fail("libams_probe.so missing: run the build first")
    lib = C.CDLL(PROBE_LIB)
    lib.ams_probe_tok_part_floats.restype = C.c_size_t
    return lib


@pytest.mark.parametrize("d,F", [(128, 128), (256, 1024), (384, 640), (1024, 4096), (2048, 5504), (4096, 11008)])
def test_tok_plan(probe, d, F):
    out = (C.c_int32 * 4)()
    Ms = list(range(65, 1300, 7)) + [2240, 4000, 9728, 19200, 32768]
    for T in (64, 100, 1300, 32768):  # a context's longest pass
        room = max(probe.ams_probe_tok_part_floats(d, k, T) for k in (d, F))
        for M in (m for m in Ms + [T] if 64 < m <= T):
            for N, K, split in ((3 * d, d, 0), (2 * F, d, 0), (d, d, 1), (d, F, 1)):
                probe.ams_probe_tok_plan(M, N, K, split, out)
                tile, splits, main_n, rest = out
                assert 0 <= tile < len(BN) and main_n % BN[tile] == 0 and 0 < main_n <= N, (M, N, K)
                assert 1 <= splits <= K // 64
                if split:
                    assert rest == -1 and main_n == N
                    assert splits == 1 or splits * M * N <= room, (M, N, K, T)
                else:
                    assert splits == 1 and (rest == -1) == (main_n == N)
                    assert rest == -1 or ((N - main_n) % BN[rest] == 0 and main_n % 32 == 0)


@pytest.mark.parametrize("M,N,K,splits", [
    (64, 4096, 4096, 1), (65, 4096, 4096, 8), (128, 4096, 11008, 16), (256, 4096, 11008, 16), (257, 4096, 11008, 8),
    (288, 4096, 4096, 8), (600, 4096, 11008, 6), (1024, 4096, 4096, 4), (2240, 1024, 1024, 2), (2240, 1024, 4096, 8),
    (2304, 4096, 11008, 2), (2305, 4096, 11008, 1), (19200, 4096, 4096, 1), (300, 384, 640, 1)])
def test_resid_splits(probe, M, N, K, splits):
    """The K ranges whose sums a residual projection adds are part of its result: they follow the
    shape alone (tiles of 256 x 256 times splits about 256, at least 8 K steps each), whatever the
    tile plan or the room for partial sums."""
    assert probe.ams_probe_tok_resid_splits(M, N, K) == splits
