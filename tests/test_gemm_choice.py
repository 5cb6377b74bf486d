"""Rules that choose the projection GEMM's blocks and the place of the LoRA
shrink (CPU: host code of the library)."""
import ctypes
import os

import pytest

from paper_2607_12422_amd import binding as b

# projections: (n-tiles, K fragments, LoRA sources, gate/up, residual) by hidden, attention width, KV width, ffn
def projections(hidden, q, kv, ffn):
    return {"qkv": ((q + 2 * kv) // 16, hidden // 32, 3, False, False), "o": (hidden // 16, q // 32, 1, False, True),
            "gate/up": (2 * ffn // 16, hidden // 32, 2, True, False), "down": (hidden // 16, ffn // 32, 1, False, True)}


@pytest.fixture(scope="module")
def rules():
    if not os.path.exists(b.LIB_PATH):
        from paper_2607_12422_amd import build
        build.build()
    lib = ctypes.CDLL(b.LIB_PATH)
    i, f = ctypes.c_int, ctypes.c_bool
    shrink = lib._ZN3pbd17gemm_shrink_tilesEiibiiiib
    shrink.argtypes, shrink.restype = [i, i, f, i, i, i, i, f], i
    return shrink


def shrink_tiles(rules, pair, lrt, proj, m_tiles):
    n_tiles, kb, nsrc, half, resid = proj
    return rules(pair, nsrc, half, lrt, n_tiles, kb, m_tiles, resid)


def test_shrink_of_a_long_k_stays_inside(rules):
    """A launch of its own walks the whole K in the few blocks it has: with 304
    fragments (ffn 9728) it costs more than the projection's own blocks lose."""
    for m_tiles in (1, 2):
        for name, proj in projections(2560, 4096, 1024, 9728).items():
            assert shrink_tiles(rules, 1, 1, proj, m_tiles) > 0, (name, m_tiles)
    # rank tiles that no instance has beside the projection
    for lrt in (0, 3):
        assert shrink_tiles(rules, 1, lrt, projections(1024, 2048, 1024, 3072)["down"], 4) == 0
