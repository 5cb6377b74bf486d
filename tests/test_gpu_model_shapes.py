"""GPU parity of bf16 models of other layer shapes than the Qwen3-0.6B one: below
hidden 256 (the skinny and the 64 x 64 GEMM with its split-K shrink), K of fewer
fragments than a block has waves, head_dim 64, one to eight query heads per KV
head, no QK RMSNorm.  Chunked prefill, draft, verify and denoising against the
float64 oracle within 2e-2, the bound of every bf16 pass.
"""
import numpy as np
import pytest

import synth
from gpu_harness import GpuRun, check_denoise, decisive
from oracle import model as om

pytestmark = pytest.mark.gpu


def shape(hidden, n_q, n_kv, head_dim, ffn, block=16, rank=16, **kw):
    return synth.QWEN3_0_6B.with_(n_layers=2, vocab=2048 + 48, hidden=hidden, n_q_heads=n_q, n_kv_heads=n_kv,
                                  head_dim=head_dim, ffn=ffn, block=block, lora_rank=rank, lora_alpha=2.0 * rank, **kw)


@pytest.mark.parametrize("cfg,batch,chunk", [
    (shape(192, 4, 2, 64, 256), 1, 0),                          # below hidden 256: few rows,
    (shape(192, 4, 2, 64, 256, rank=48), 4, 30),                # 68 rows,
    (shape(128, 2, 2, 64, 320, rank=64), 9, 40),                # 153 rows: fp16 operands, shrink over K slices
    (shape(64, 1, 1, 128, 64), 10, 100),                        # two fragments of K everywhere
    (shape(256, 1, 1, 64, 64, rank=64), 3, 40),                 # o and down of two fragments
    (shape(256, 1, 1, 64, 64, rank=32), 17, 20),                # ... in 289 rows
    (shape(320, 5, 1, 64, 960, block=15), 5, 33),               # head_dim 64: five tiles of query rows
    (shape(512, 8, 2, 64, 1536, rank=8), 20, 64),
    (shape(512, 2, 2, 128, 768), 1, 70),                        # one query head per KV head
    (shape(512, 2, 2, 128, 768, block=31), 4, 70),
    (shape(384, 6, 2, 128, 512, rank=32), 3, 50),               # three
    (shape(512, 8, 2, 128, 1024, rank=64), 2, 0),               # four
    (shape(512, 8, 1, 128, 1024, block=9), 5, 45),              # eight
    (shape(1024, 16, 8, 128, 3072, qk_norm=False), 1, 90),      # no QK RMSNorm
    (shape(1024, 16, 8, 128, 3072, qk_norm=False), 3, 64),
    (shape(512, 8, 4, 64, 1536, qk_norm=False), 3, 64),
])
def test_model_shapes_match_oracle(cfg, batch, chunk):
    w = synth.make_weights(cfg, 97)
    rng = np.random.Generator(np.random.PCG64(8))
    lengths = [int(x) for x in rng.integers(1, 120, size=batch)]
    prompts = synth.make_prompts(cfg, lengths, 10)
    g = GpuRun(cfg, w, max_batch=batch, max_seq=max(lengths) + 3 * cfg.width, prefill_chunk=chunk)
    first = g.prefill(prompts)
    d, dlg = g.draft()
    v, vlg = g.verify(d)
    dn, conf, fixed, nlg = g.denoise(2)
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in sorted({0, batch // 2, batch - 1}):
        st = om.prefill(m, prompts[b])
        st.anchor = int(first[b])
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
