"""GPU parity of the K-split and LDS-tiled projection GEMMs (bf16 passes; here of
more than 32 rows, test_gpu_gemm_instances.py has the blocks that these do not
reach) at the edges of their blocks: one row past an m-tile, a last block with missing
m-tiles, a vocabulary whose last block has missing tiles; LoRA ranks whose
shrink runs inside the projection (one, two and four A tiles) and as a launch
of its own (three; four with two sources); the softmax partials of its LM head
(denoising confidence).  Draft and verify logits against the float64 oracle
within 2e-2, the bound of every bf16 pass.
"""
import numpy as np
import pytest

import synth
from gpu_harness import GpuRun, check_denoise, decisive
from oracle import model as om

pytestmark = pytest.mark.gpu

SHAPE = synth.QWEN3_0_6B.with_(n_layers=1, vocab=4096 + 16)


@pytest.mark.parametrize("batch,block,rank,max_batch", [
    (3, 10, 16, 3),      # 33 rows: three m-tiles, one live row in the last
    (3, 16, 32, 3),      # 51 rows
    (5, 16, 48, 5),      # 85 rows: six m-tiles, three shrink tiles per source
    (7, 16, 64, 7),      # 119 rows: value + residual operands
    (8, 16, 16, 8),      # 136 rows: fp16 operands, nine m-tiles
    (8, 16, 48, 8),
    (11, 24, 64, 11),    # 275 rows: fp16 operands, 18 m-tiles
    (21, 15, 8, 21),     # 336 rows: the LM head on the other GEMM
    (5, 8, 32, 40),      # 45 rows in a context sized for fp16 passes
])
def test_rows_and_ranks_match_oracle(batch, block, rank, max_batch):
    cfg = SHAPE.with_(block=block, lora_rank=rank, lora_alpha=2.0 * rank)
    w = synth.make_weights(cfg, 77)
    rng = np.random.Generator(np.random.PCG64(5))
    lengths = [int(x) for x in rng.integers(1, 60, size=batch)]
    prompts = synth.make_prompts(cfg, lengths, 6)
    g = GpuRun(cfg, w, max_batch=max_batch, max_seq=128)
    g.prefill(prompts)
    anchors = g.anchor.cpu().numpy()
    d, dlg = g.draft()
    v, vlg = g.verify(d)
    dn, conf, fixed, nlg = g.denoise(2)
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in sorted({0, batch // 2, batch - 1}):
        st = om.prefill(m, prompts[b])
        st.anchor = int(anchors[b])
        ref_d, ref_dl = om.draft(m, st)
        assert np.abs(dlg[b].cpu().numpy() - ref_dl).max() <= 2e-2
        ok = decisive(ref_dl[1:], 2e-2, exclude=cfg.mask_id)
        assert np.array_equal(d[b].cpu().numpy()[ok], ref_d[ok])
        ref_p, ref_vl, _, _ = om.verify(m, st, d[b].cpu().numpy())
        assert np.abs(vlg[b].cpu().numpy() - ref_vl).max() <= 2e-2
        ok = decisive(ref_vl, 2e-2)
        assert np.array_equal(v[b].cpu().numpy()[ok], ref_p[ok])
        check_denoise(m, st, dn[b].cpu().numpy(), conf[b].cpu().numpy(), fixed[b].cpu().numpy(), nlg[b].cpu().numpy(),
                      2, 2e-2, what=f"sequence {b}")
    g.close()


@pytest.mark.parametrize("chunk", [33, 64, 129])
def test_prefill_chunks_match_oracle(chunk):
    cfg = SHAPE
    w = synth.make_weights(cfg, 78)
    lengths = [140, 33]
    prompts = synth.make_prompts(cfg, lengths, 7)
    g = GpuRun(cfg, w, max_batch=2, max_seq=192, prefill_chunk=chunk)
    g.prefill(prompts)
    anchors = g.anchor.cpu().numpy()
    v, vlg = g.verify(g.i32(np.full((2, cfg.block), 9)))
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in range(2):
        st = om.prefill(m, prompts[b])
        st.anchor = int(anchors[b])
        _, ref, _, _ = om.verify(m, st, np.full(cfg.block, 9))
        assert np.abs(vlg[b].cpu().numpy() - ref).max() <= 2e-2
    g.close()


@pytest.mark.parametrize("batch,block,rank", [
    (16, 15, 48),        # 256 rows: 4 x 8 blocks, three shrink tiles per source (one and a half products)
    (25, 15, 64),        # 400 rows: 4 x 8 and 8 x 8, a last row block with one m-tile
    (45, 17, 8),         # 810 rows: 8 x 8 and 10 x 8, a last m-tile with ten rows
    (32, 32, 64),        # 1056 rows: 10 x 8 and 8 x 16
])
def test_lds_blocks_match_oracle(batch, block, rank):
    """Rows enough for the LDS-tiled blocks; a vocabulary that leaves the LM
    head's last block incomplete.  Sampled sequences against the oracle."""
    cfg = SHAPE.with_(block=block, lora_rank=rank, lora_alpha=2.0 * rank)
    w = synth.make_weights(cfg, 79)
    rng = np.random.Generator(np.random.PCG64(6))
    lengths = [int(x) for x in rng.integers(1, 60, size=batch)]
    prompts = synth.make_prompts(cfg, lengths, 6)
    g = GpuRun(cfg, w, max_batch=batch, max_seq=160)
    g.prefill(prompts)
    anchors = g.anchor.cpu().numpy()
    d, dlg = g.draft()
    v, vlg = g.verify(d)
    dn, conf, fixed, nlg = g.denoise(2)
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in (0, batch - 1):
        st = om.prefill(m, prompts[b])
        st.anchor = int(anchors[b])
        _, ref_dl = om.draft(m, st)
        assert np.abs(dlg[b].cpu().numpy() - ref_dl).max() <= 2e-2
        ref_p, ref_vl, _, _ = om.verify(m, st, d[b].cpu().numpy())
        assert np.abs(vlg[b].cpu().numpy() - ref_vl).max() <= 2e-2
        ok = decisive(ref_vl, 2e-2)
        assert np.array_equal(v[b].cpu().numpy()[ok], ref_p[ok])
        check_denoise(m, st, dn[b].cpu().numpy(), conf[b].cpu().numpy(), fixed[b].cpu().numpy(), nlg[b].cpu().numpy(),
                      2, 2e-2, what=f"sequence {b}")
    g.close()


@pytest.mark.parametrize("batch,chunk,lengths", [
    (1, 1000, [2000]),           # 1000 rows of value + residual operands: 8 x 8 and 8 x 12
    (4, 1024, [1100, 70, 1024, 5]),   # 4096 rows, m-blocks shared out among the XCDs
])
def test_long_prefill_chunks_match_oracle(batch, chunk, lengths):
    cfg = SHAPE
    w = synth.make_weights(cfg, 80)
    prompts = synth.make_prompts(cfg, lengths, 7)
    g = GpuRun(cfg, w, max_batch=batch, max_seq=max(lengths) + 64, prefill_chunk=chunk)
    first = g.prefill(prompts)
    v, vlg = g.verify(g.i32(np.full((batch, cfg.block), 9)))
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in range(batch):
        st = om.prefill(m, prompts[b])
        st.anchor = int(first[b])
        _, ref, _, _ = om.verify(m, st, np.full(cfg.block, 9))
        assert np.abs(vlg[b].cpu().numpy() - ref).max() <= 2e-2
    g.close()
