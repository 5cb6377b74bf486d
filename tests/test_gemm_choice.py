"""Rules that choose the projection GEMM's blocks and the place of the LoRA
shrink (CPU: host code of the library)."""
import ctypes
import os

import pytest

import test_gpu_gemm_instances as instances
import test_gpu_ksplit_gemm as ksplit
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
    choice = lib._ZN3pbd11gemm_choiceEiiiiibbPi
    choice.argtypes, choice.restype = [i, i, i, i, i, f, f, ctypes.POINTER(i)], i
    return shrink, choice


def shrink_tiles(rules, pair, lrt, proj, m_tiles):
    n_tiles, kb, nsrc, half, resid = proj
    return rules[0](pair, nsrc, half, lrt, n_tiles, kb, m_tiles, resid)


def block(rules, pair, st, n_tiles, kb, m_tiles, argmax, resid):
    """(operands, LDS block, m-tiles, n-tiles, waves, shrink tiles, LM head) of a launch."""
    out = (ctypes.c_int * 4)()
    assert rules[1](pair, st, n_tiles, kb, m_tiles, argmax, resid, out), (pair, st, n_tiles, kb, m_tiles, argmax)
    return (pair, *out, st, argmax)


def layer_blocks(rules, projs, pair, m_tiles, lrt):
    """Blocks (and whether u comes from a launch before) of one layer's launches."""
    got = set()
    if m_tiles < 3 and lrt > m_tiles:           # the skinny GEMM's
        return got
    for proj in projs.values():
        n_tiles, kb, nsrc, _, resid = proj
        st = shrink_tiles(rules, pair, lrt, proj, m_tiles) if lrt else 0
        got.add((*block(rules, pair, st, n_tiles, kb, m_tiles, False, resid), lrt > 0 and st == 0))
        if lrt and not st:
            got.add((*block(rules, pair, 0, nsrc * lrt, kb, m_tiles, False, False), False))
    return got


def step_blocks(rules, projs, batch, width, rank, max_batch, vocab):
    """Blocks of a draft (adapter on) and a verify (off)."""
    rows = batch * width
    m_tiles = (rows + 15) // 16
    pair = 0 if max_batch * width >= 128 and m_tiles >= 8 else 1
    got = layer_blocks(rules, projs, pair, m_tiles, (rank + 15) // 16) | layer_blocks(rules, projs, pair, m_tiles, 0)
    if m_tiles >= 3:
        got.add((*block(rules, pair, 0, vocab // 16, projs["qkv"][1], m_tiles, True, False), False))
    return got


def params(test):
    return next(m for m in test.pytestmark if m.name == "parametrize").args[1]


def test_shrink_of_a_long_k_stays_inside(rules):
    """A launch of its own walks the whole K in the few blocks it has: with 304
    fragments (ffn 9728) it costs more than the projection's own blocks lose."""
    for m_tiles in (1, 2):
        for name, proj in projections(2560, 4096, 1024, 9728).items():
            assert shrink_tiles(rules, 1, 1, proj, m_tiles) > 0, (name, m_tiles)
    # rank tiles that no instance has beside the projection
    for lrt in (0, 3):
        assert shrink_tiles(rules, 1, lrt, projections(1024, 2048, 1024, 3072)["down"], 4) == 0


def test_gpu_tests_run_every_block_of_the_qwen_layer(rules):
    """Every block (and place of the shrink) that a step of 1 to 32 sequences or
    a prefill chunk of the Qwen3-0.6B layer can take is run by a parity test."""
    q = projections(1024, 2048, 1024, 3072)
    need, tested = {}, set()
    for batch in range(1, 33):
        for width in range(1, 34):
            for rank in (16, 32, 48, 64):
                for k in step_blocks(rules, q, batch, width, rank, batch, instances.FULL):
                    need.setdefault(k, (batch, width, rank))
    for rows in range(1, 4097):
        if rows <= 1024 or rows % 8 == 0:       # chunks of up to 1024 rows of several sequences
            for k in layer_blocks(rules, q, 1, (rows + 15) // 16, 0):
                need.setdefault(k, rows)
    for batch, blk, rank, max_batch in params(ksplit.test_rows_and_ranks_match_oracle):
        tested |= step_blocks(rules, q, batch, blk + 1, rank, max_batch, ksplit.SHAPE.vocab)
    for batch, blk, rank in params(ksplit.test_lds_blocks_match_oracle):
        tested |= step_blocks(rules, q, batch, blk + 1, rank, batch, ksplit.SHAPE.vocab)
    for batch, blk, rank, vocab in instances.STEPS:
        tested |= step_blocks(rules, q, batch, blk + 1, rank, batch, vocab)
    chunks = [(2, c) for c in params(ksplit.test_prefill_chunks_match_oracle)] + instances.PREFILLS
    chunks += [(batch, c) for batch, c, _ in params(ksplit.test_long_prefill_chunks_match_oracle)]
    for batch, chunk in chunks:
        tested |= layer_blocks(rules, q, 1, (batch * chunk + 15) // 16, 0)
    missing = {k: where for k, where in need.items() if k not in tested}
    assert not missing, missing
