"""GPU parity of the projection GEMM blocks that passes of the Qwen3-0.6B layer
take and the tests of test_gpu_ksplit_gemm.py do not reach: draft, verify and
denoising (argmax and softmax partials) against the float64 oracle within 2e-2,
the bound of every bf16 pass.  test_gemm_choice.py checks (on the CPU) that both
files together run every block that such passes can take.
"""
import numpy as np
import pytest

import synth
from gpu_harness import GpuRun, check_denoise, decisive
from oracle import model as om

pytestmark = pytest.mark.gpu

SMALL = 4096 + 16         # a last LM-head block with missing tiles
FULL = 151936             # 9496 tiles: half of the last 16-tile block missing

STEPS = [
    # (sequences, block, rank, vocabulary)
    (1, 16, 32, SMALL),       # two m-tiles: four shrink tiles beside gate/up
    (1, 32, 48, SMALL),       # three m-tiles, shrink launches of three tiles
    (3, 15, 16, FULL),        # LM heads of three,
    (4, 16, 32, FULL),        # five
    (6, 16, 64, FULL),        # and seven m-tiles of value + residual operands
    (8, 16, 64, FULL),        # ... and of nine of fp16
    (2, 24, 64, SMALL),       # four m-tiles
    (3, 32, 16, SMALL),       # seven
    (13, 4, 16, SMALL),       # five, five rows a sequence
    (26, 4, 32, SMALL),       # 130 rows: fp16, two rows in the last m-tile
    (26, 4, 64, SMALL),
    (4, 31, 16, SMALL),       # 128 rows: eight m-tiles, all full
    (4, 31, 32, SMALL),
    (4, 31, 48, SMALL),
    (4, 31, 64, SMALL),
    (6, 32, 16, SMALL),       # 198 rows: 13 m-tiles
    (6, 32, 32, SMALL),
    (6, 32, 64, SMALL),
    (29, 8, 48, SMALL),       # 261 rows: 17 m-tiles
    (25, 32, 48, SMALL),      # 825 rows: 52
]
PREFILLS = [
    # (sequences, prompt rows per pass)
    (1, 322),
    (2, 643),
    (2, 706),
]


@pytest.mark.parametrize("batch,block,rank,vocab", STEPS)
def test_steps_match_oracle(batch, block, rank, vocab):
    cfg = synth.QWEN3_0_6B.with_(n_layers=1, vocab=vocab, block=block, lora_rank=rank, lora_alpha=2.0 * rank)
    w = synth.make_weights(cfg, 95)
    rng = np.random.Generator(np.random.PCG64(7))
    prompts = synth.make_prompts(cfg, [int(x) for x in rng.integers(1, 40, size=batch)], 8)
    g = GpuRun(cfg, w, max_batch=batch, max_seq=128)
    g.prefill(prompts)
    anchors = g.anchor.cpu().numpy()
    d, dlg = g.draft()
    v, vlg = g.verify(d)
    dn, conf, fixed, nlg = g.denoise(2)
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in sorted({0, batch - 1}):
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


@pytest.mark.parametrize("batch,chunk", PREFILLS)
def test_prefill_chunks_match_oracle(batch, chunk):
    cfg = synth.QWEN3_0_6B.with_(n_layers=1, vocab=SMALL)
    w = synth.make_weights(cfg, 96)
    prompts = synth.make_prompts(cfg, [chunk - 3 * b for b in range(batch)], 9)
    g = GpuRun(cfg, w, max_batch=batch, max_seq=chunk + 64, prefill_chunk=chunk)
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
