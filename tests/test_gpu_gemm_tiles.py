"""A row's result does not depend on how many rows are computed with it: the projections pick their tiles (and, for 16-bit
operands, split a product into two launches) by the row count, so a sequence alone, in a small batch and in a large one
meets different kernels.  Every batch is compared with the same rows of the largest one bit for bit, and the largest one
with the fp64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2601_15013_amd import binding, harness, synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

# row counts around the edges of the tiles (16, 32, 64, 128, 256) and of the chip's rounds of workgroups
ROWS_16 = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 513, 800, 1100, 2070, 2200, 4500, 8300, 9000]
ROWS_F32 = [1, 15, 16, 17, 31, 33, 63, 64, 65, 200, 513, 1100, 4500]

SMALL = synth.ModelConfig("tiles16", 1, 256, 4, 2, 128, 320, 512, "bf16", max_pos=64)              # widths that are odd multiples of 128
WIDE = synth.ModelConfig("tiles16w", 1, 1024, 16, 8, 128, 3072, 512, "bf16", max_pos=64)
F32 = synth.ModelConfig("tiles32", 1, 132, 6, 2, 44, 96, 300, "f32", max_pos=64)                 # K and widths not multiples of the tiles


def nodedup(model, tok, lens):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    run = harness.Runner(model, int(cu[-1]), len(lens))
    y = run.forward_nodedup(torch.from_numpy(tok[: cu[-1]]).cuda(), torch.from_numpy(cu).cuda(), int(max(lens)))
    assert run.status() == 0
    return y.cpu().numpy()


@pytest.mark.parametrize("cfg,compute,hilo,tol", [(SMALL, None, -1, 2e-2), (SMALL, "bf16", 1, 0.5), (WIDE, None, -1, 2e-2),
                                                  (WIDE, None, 1, 2e-2), (F32, None, 0, 1e-4)])
def test_rows_do_not_depend_on_the_batch(cfg, compute, hilo, tol):
    # tolerances: those of the parity tests (fp32 1e-4, fp16 operands 2e-2); bf16 operands carry no parity claim
    rows = ROWS_F32 if cfg.dtype == "f32" else ROWS_16
    w = synth.SynthWeights(cfg, 77)
    rng = np.random.default_rng(5)
    tok = rng.integers(0, cfg.vocab, size=max(rows), dtype=np.int32)
    model = harness.upload_model(w, compute_dtype=compute, hilo_layers=hilo)
    try:
        def lens(n):                       # sequences of 23 tokens, the last one shorter: a prefix of the larger batches
            return [23] * (n // 23) + ([n % 23] if n % 23 else [])
        full = nodedup(model, tok, lens(max(rows)))
        for n in rows[:-1]:
            assert np.array_equal(nodedup(model, tok, lens(n)), full[:n]), n
    finally:
        model.close()
    pick = np.array([0, 1, len(lens(max(rows))) // 2, len(lens(max(rows))) - 1])
    cu = np.concatenate([[0], np.cumsum(lens(max(rows)))]).astype(np.int32)
    from oracle import forward as oracle_forward
    for s in pick:
        t = tok[cu[s]:cu[s + 1]]
        ref = oracle_forward.forward_nodedup(cfg, w.embed, w.layers, w.gf, t, np.array([0, len(t)], dtype=np.int32))
        got = full[cu[s]:cu[s + 1]]
        assert np.max(np.abs(got - ref)) <= tol * np.sqrt(np.mean(ref * ref)), s


@pytest.mark.parametrize("own,pads", [(164, (64, 512)), (163, (1000,))])
def test_padding_of_a_compact_space_whose_products_are_split(own, pads):
    # 8230 or 8180 unique rows: the padded products are cut at 8192 rows, before the last representative and among the padding;
    # the output projection of the three-kernel path reads its rows through I_gather on both sides of the cut
    rng = np.random.default_rng(own)
    prefix = rng.integers(0, 512, 30, dtype=np.int32)
    seqs = [np.concatenate([prefix, [b], rng.integers(0, 512, own - 1)]).astype(np.int32) for b in range(50)]
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum([len(x) for x in seqs])]).astype(np.int32)).cuda()
    tok = torch.from_numpy(np.concatenate(seqs)).cuda()
    model = harness.upload_model(synth.SynthWeights(dataclasses.replace(WIDE, max_pos=256), 79))
    try:
        run = harness.Runner(model, tok.numel(), len(seqs))
        maps = run.build_index(tok, cu)
        assert maps[3] == 30 + 50 * own
        longest = 30 + own
        plain = run.forward_nodedup(tok, cu, longest)
        for fused in (False, True):
            for pad in (0,) + pads:
                y = run.forward(tok, cu, longest, maps, force_dedup=True, fused_attention=fused, pad_compact_to=pad)
                assert run.status() == 0
                assert torch.equal(y, plain), (pad, fused)
    finally:
        model.close()


@pytest.mark.parametrize("n_rows", [1, 33, 300])
def test_lm_head_rows_do_not_depend_on_their_number(n_rows):
    cfg = synth.ModelConfig("tileshead", 1, 256, 2, 2, 128, 128, 1408, "bf16", max_pos=64)
    w = synth.SynthWeights(cfg, 78)
    model = harness.upload_model(w, lm_head_mode=1)
    try:
        hidden = torch.from_numpy(np.random.default_rng(1).standard_normal((700, cfg.d)).astype(np.float32)).cuda()
        ws = binding.alloc_workspace(binding.radix_lm_head_workspace_bytes(model, 700))
        full = binding.radix_lm_head(model, hidden, None, ws).cpu().numpy()
        some = binding.radix_lm_head(model, hidden[:n_rows].contiguous(), None, ws).cpu().numpy()
        assert np.array_equal(some, full[:n_rows])
        h = hidden[:n_rows].cpu().numpy().astype(np.float16).astype(np.float64)
        ref = h @ np.asarray(w.embed, dtype=np.float64).T
        # operands are the exact fp16 values up to weights below 2^-17; fp32 accumulation over 256 terms
        assert np.max(np.abs(some - ref)) <= 256 * 2.0 ** -23 * np.max(np.abs(h) @ np.abs(np.asarray(w.embed, dtype=np.float64)).T)
    finally:
        model.close()


@pytest.mark.parametrize("B", [1, 15, 16, 17, 18, 63, 257, 1025])
@pytest.mark.parametrize("with_pos", [False, True])
def test_index_first_round_over_the_chip(B, with_pos):
    # on both sides of where the first round of comparisons gets a launch of its own (by the amount to compare): shared
    # prefixes longer than a wavefront's stride, empty sequences in front and between, duplicates, whole prefixes
    rng = np.random.default_rng(B)
    base = rng.integers(0, 50, size=1300, dtype=np.int32)
    seqs = []
    for b in range(B):
        kind = b % 7
        cut = int(rng.integers(0, 1300))
        if b == 0 and B > 2 or kind == 5:
            seqs.append(base[:0])
        elif kind in (0, 1):
            seqs.append(np.concatenate([base[:cut], rng.integers(0, 50, size=int(rng.integers(0, 40)), dtype=np.int32)]))
        elif kind == 2:
            seqs.append(base[:cut])
        elif kind == 3:
            seqs.append(base.copy())
        else:
            seqs.append(np.concatenate([base[:1111], rng.integers(0, 3, size=int(rng.integers(0, 9)), dtype=np.int32)]))
    cu = np.concatenate([[0], np.cumsum([len(s) for s in seqs])]).astype(np.int32)
    tok = np.concatenate(seqs).astype(np.int32)
    pos = None
    if with_pos:
        pos = np.concatenate([np.arange(len(s)) + (3 if b % 11 == 10 else 0) for b, s in enumerate(seqs)]).astype(np.int32)
    U.assert_index_parity(tok, cu, pos)


@pytest.mark.parametrize("B", [4095, 4096, 4097, 9000])
def test_index_table_in_lds_and_in_memory(B):
    # around the number of sequences whose grouping table still fits LDS: many followers leave a leader at one depth,
    # with few (collisions of equal keys) and with many (collisions of slots) distinct tokens
    rng = np.random.default_rng(B)
    seqs = [np.concatenate([[7, 7], rng.integers(0, 3 if b % 2 else 100000, size=int(rng.integers(0, 4)))]).astype(np.int32)
            for b in range(B)]
    cu = np.concatenate([[0], np.cumsum([len(s) for s in seqs])]).astype(np.int32)
    U.assert_index_parity(np.concatenate(seqs), cu)


@pytest.mark.parametrize("B", [17, 300])
def test_malformed_cu_seqlens_leaves_the_maps_untouched(B):
    n = 10 * B
    cu = np.arange(B + 1, dtype=np.int32) * 10
    cu[B // 2] = n + 5
    tok = torch.zeros(n, dtype=torch.int32, device="cuda")
    I_s = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    I_g = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    n_dev = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(B))
    with pytest.raises(Exception):
        binding.radix_build_index(tok, None, torch.from_numpy(cu).cuda(), ws, I_s, I_g, n_dev)
    assert int(n_dev.item()) == 0 and bool((I_s == -7).all()) and bool((I_g == -7).all())
