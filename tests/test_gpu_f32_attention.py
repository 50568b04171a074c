"""fp32 attention through the index maps: the deduplicated forward gives the bits of the three-kernel sequence and of the plain
forward, around the batches of value rows (16), the chunks of keys (64), heads of at most and of more than 64, and with padding."""
import numpy as np
import pytest
import torch

from paper_2601_15013_amd import harness, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [36, 64, 68, 128])
@pytest.mark.parametrize("prefix,own", [(1, 1), (3, 12), (8, 8), (15, 2), (47, 17), (63, 2), (64, 1), (100, 93)])
def test_same_bits_in_every_mode(head_dim, prefix, own):
    cfg = synth.ModelConfig("f32att", 2, 132, 4, 2, head_dim, 96, 300, "f32", max_pos=512)
    weights = synth.SynthWeights(cfg, head_dim)
    b = synth.shared_prefix_batch(prefix * 7 + own, 5, prefix, own, own + 3, cfg.vocab)
    model = harness.upload_model(weights)
    try:
        run = harness.Runner(model, b.N, b.B)
        tok, cu = harness.upload_batch(b)
        maps = run.build_index(tok, cu)
        assert maps[3] == b.expected_n_compact < b.N
        plain = run.forward_nodedup(tok, cu, b.max_seqlen).clone()
        for kw in ({}, {"fused_attention": False}, {"pad_compact_to": 64}):
            y = run.forward(tok, cu, b.max_seqlen, maps, force_dedup=True, **kw).clone()
            assert torch.equal(y, plain), kw
        assert run.status() == 0
    finally:
        model.close()


def test_a_map_entry_out_of_range_is_clamped_and_reported():
    cfg = synth.TINY
    b = synth.shared_prefix_batch(3, 4, 20, 5, 9, cfg.vocab)
    model = harness.upload_model(synth.SynthWeights(cfg, 1))
    try:
        run = harness.Runner(model, b.N, b.B)
        tok, cu = harness.upload_batch(b)
        I_s, I_g, n_dev, n = run.build_index(tok, cu)
        for i, value in ((b.N - 1, n), (2, -1)):
            bad = I_s.clone()
            bad[i] = value
            run.forward(tok, cu, b.max_seqlen, (bad, I_g, n_dev, n), force_dedup=True)
            assert run.status() == -7
    finally:
        model.close()
