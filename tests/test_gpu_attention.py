"""GPU parity of the attention of draft and verify passes (bf16, head_dim 128)
at the edges of its work split: one to five 16-row query tiles per KV head with
a full or a nearly empty last tile, prefixes around the 16-key blocks, the
32-key stages and the depth of their ring, splits of one block, of an odd
number of blocks and automatic ones, a block of two stages.  Logits against the
float64 oracle within 2e-2, the bound of every bf16 pass.
"""
import numpy as np
import pytest

import synth
from gpu_harness import GpuRun, decisive
from oracle import model as om

pytestmark = pytest.mark.gpu

SHAPE = synth.QWEN3_0_6B.with_(n_layers=2, vocab=4096)


@pytest.mark.parametrize("block,lengths,kps", [
    (1, [1, 15, 16], 0),            # one tile, four live rows; less than a stage
    (7, [17, 31, 300], 48),         # one full tile; splits of a stage and a half
    (8, [32, 33, 97], 16),          # two tiles, two rows in the last; splits of one block
    (15, [63, 64, 65], 0),          # two full tiles
    (16, [95, 129, 700], 0),        # three tiles, two rows in the last
    (16, [1, 160, 161], 80),        # ... splits of five blocks
    (23, [48, 127, 257], 112),      # three full tiles
    (24, [2, 96, 511], 0),          # four tiles
    (31, [128, 130, 400], 176),     # four full tiles, a block of exactly 32 keys
    (32, [16, 225, 513], 0),        # five tiles, a block of two stages
])
def test_tiles_and_splits_match_oracle(block, lengths, kps):
    cfg = SHAPE.with_(block=block)
    w = synth.make_weights(cfg, 91)
    prompts = synth.make_prompts(cfg, lengths, 8)
    g = GpuRun(cfg, w, max_batch=3, max_seq=max(lengths) + 2 * cfg.width + 5)
    g.eng.pbd_set_attn_keys_per_split(kps)
    g.prefill(prompts)
    anchors = g.anchor.cpu().numpy()
    d, dlg = g.draft()
    v, vlg = g.verify(d)
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in range(3):
        st = om.prefill(m, prompts[b])
        st.anchor = int(anchors[b])
        _, ref_dl = om.draft(m, st)
        assert np.abs(dlg[b].cpu().numpy() - ref_dl).max() <= 2e-2
        ref_p, ref_vl, _, _ = om.verify(m, st, d[b].cpu().numpy())
        assert np.abs(vlg[b].cpu().numpy() - ref_vl).max() <= 2e-2
        ok = decisive(ref_vl, 2e-2)
        assert np.array_equal(v[b].cpu().numpy()[ok], ref_p[ok])
    g.close()
