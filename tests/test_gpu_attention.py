"""GPU parity of the attention of draft and verify passes and of prefill chunks
(bf16, head_dim 128) at the edges of its work split: one to five 16-row query tiles per KV head with
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
from paper_2607_12422_amd import binding

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


@pytest.mark.parametrize("batch,block,max_seq,keys,mode", [
    (1, 16, 802, 256, 1),           # one sequence, up to three tiles: one work-group per tile
    (1, 7, 300, 256, 1),
    (1, 32, 802, 256, 0),           # ... five tiles, few splits: one work-group per KV head
    (1, 32, 2100, 256, 1),          # ... and nine of them
    (2, 16, 802, 256, 0),           # more sequences: one work-group per KV head
    (5, 16, 8300, 512, 0),          # 5 x 8 x 33 work items of 256 keys are too many
])
def test_automatic_layout_is_the_documented_one(batch, block, max_seq, keys, mode):
    """The automatic keys per split and layout give bitwise what the values
    that pbd.h names for them give."""
    cfg = SHAPE.with_(n_layers=1, block=block, lora_rank=32, lora_alpha=64.0)
    w = synth.make_weights(cfg, 93)
    g = GpuRun(cfg, w, max_batch=batch, max_seq=max_seq)
    g.prefill(synth.make_prompts(cfg, [260 - 7 * b for b in range(batch)], 10))
    _, automatic = g.draft()
    g.eng.pbd_set_attn_keys_per_split(keys)
    g.eng.pbd_set_attn_query_split(mode)
    _, named = g.draft()
    assert g.status() == 0
    assert bool((automatic == named).all())
    g.eng.pbd_set_attn_query_split(1 - mode)
    _, other = g.draft()
    assert not bool((other == named).all())
    g.close()


@pytest.mark.parametrize("block,batch", [(0, 6), (7, 4), (16, 4), (31, 3)])
def test_one_reference_maximum_is_no_less_precise(block, batch):
    """k_attn_rows (layout 0) keeps one reference maximum per query row and
    split, k_attn (layout 1) four: the weights that bf16 holds exactly are those
    at a maximum.  On the same cache, the error of the verify's logits against
    float64 (2-norm over all seeds) must not be larger than k_attn's by more
    than twice the standard error of their ratio over the seeds."""
    cfg = SHAPE.with_(n_layers=1, block=block)
    err = np.zeros((2, 8))
    for seed in range(err.shape[1]):
        w = synth.make_weights(cfg, 300 + seed)
        prompts = synth.make_prompts(cfg, [250 - 9 * b for b in range(batch)], 400 + seed)
        g = GpuRun(cfg, w, max_batch=batch, max_seq=300)
        first = g.prefill(prompts)
        drafts = np.random.Generator(np.random.PCG64(seed)).integers(0, cfg.vocab - 1, size=(batch, max(block, 1)))
        got = []
        for mode in (0, 1):
            g.eng.pbd_set_attn_query_split(mode)
            _, lg = g.verify(g.i32(drafts[:, :block] if block else drafts))
            got.append(lg.cpu().numpy().astype(np.float64))
        assert g.status() == 0
        g.close()
        m = om.OracleModel(w)
        for b in range(batch):
            st = om.prefill(m, prompts[b])
            st.anchor = int(first[b])
            _, ref, _, _ = om.verify(m, st, drafts[b, :block])
            for mode in (0, 1):
                err[mode, seed] += ((got[mode][b] - ref) ** 2).sum()
    err = np.sqrt(err)
    ratio = np.log(err[0] / err[1])
    print(f"block {block}: rows / one-tile {np.exp(ratio.mean()):.4f} +- {ratio.std(ddof=1) / len(ratio) ** 0.5:.4f}")
    assert ratio.mean() <= 2 * ratio.std(ddof=1) / len(ratio) ** 0.5


@pytest.mark.parametrize("chunk,lengths", [
    (1, [3, 5, 1]),                 # one row per pass
    (31, [40, 1, 62]),              # a row block over both query heads
    (64, [64, 65, 129]),            # one block per head; a sequence of one chunk
    (100, [350, 7, 100]),           # a short sequence ends before the last chunks
    (300, [700, 301, 5]),           # several stages, causal rows in the last ones
    (513, [513, 512, 130]),         # a last block with two rows
])
def test_prefill_chunks_match_oracle(chunk, lengths):
    cfg = SHAPE
    w = synth.make_weights(cfg, 92)
    prompts = synth.make_prompts(cfg, lengths, 9)
    g = GpuRun(cfg, w, max_batch=3, max_seq=max(lengths) + 2 * cfg.width, prefill_chunk=chunk)
    first = g.prefill(prompts)
    v, vlg = g.verify(g.i32(np.full((3, cfg.block), 9)))
    assert g.status() == 0
    m = om.OracleModel(w)
    for b in range(3):
        st = om.prefill(m, prompts[b])
        st.anchor = int(first[b])
        _, ref, _, _ = om.verify(m, st, np.full(cfg.block, 9))
        assert np.abs(vlg[b].cpu().numpy() - ref).max() <= 2e-2
    g.close()


@pytest.mark.parametrize("keys,splits", [(0, False), (2048, True)])
def test_keys_per_split_reach_the_prefill(keys, splits):
    """Keys per split set by the caller split a prefill chunk's attention too
    (there are partials to merge); automatic, a short prompt's is not split."""
    cfg = SHAPE
    w = synth.make_weights(cfg, 94)
    prompts = synth.make_prompts(cfg, [600], 11)
    g = GpuRun(cfg, w, max_batch=1, max_seq=700, prefill_chunk=600)
    g.eng.pbd_set_attn_keys_per_split(keys)
    g.eng.pbd_profile_enable(True)
    first = g.prefill(prompts)
    _, merges = g.eng.pbd_profile_read(binding.KCLASSES.index("combine"))
    g.eng.pbd_profile_enable(False)
    assert (merges == cfg.n_layers) if splits else (merges == 0)
    v, vlg = g.verify(g.i32(np.full((1, cfg.block), 9)))
    assert g.status() == 0
    m = om.OracleModel(w)
    st = om.prefill(m, prompts[0])
    st.anchor = int(first[0])
    _, ref, _, _ = om.verify(m, st, np.full(cfg.block, 9))
    assert np.abs(vlg[0].cpu().numpy() - ref).max() <= 2e-2
    g.close()
