"""Forwards over very many sequences: what a forward does per sequence (checking cu_seqlens, finding the sequence of a token)
must not outweigh the rows, and must be right at the sizes where the search takes another step."""
import numpy as np
import pytest
import torch

from paper_2601_15013_amd import harness, synth

pytestmark = pytest.mark.gpu

CFG = synth.ModelConfig("many", 1, 128, 1, 1, 128, 64, 512, "bf16", max_pos=512)


@pytest.fixture(scope="module")
def model():
    m = harness.upload_model(synth.SynthWeights(CFG, 5), hilo_layers=-1)
    yield m
    m.close()


def forward(model, lens, pos=None, max_seqlen=None):
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    n = int(sum(lens))
    tok = torch.from_numpy(np.random.default_rng(1).integers(0, CFG.vocab, n, dtype=np.int32)).cuda()
    run = harness.Runner(model, n, len(lens))
    pos_t = None if pos is None else torch.from_numpy(pos.astype(np.int32)).cuda()
    longest = int(max(lens)) if max_seqlen is None else max_seqlen
    return run, lambda out=None: run.forward_nodedup(tok, cu, longest, pos=pos_t, out=out)


@pytest.mark.parametrize("B", [1, 2, 63, 64, 65, 127, 4095, 4096, 4097, 8191, 8193, 65535])
def test_default_positions_are_the_offsets_in_the_sequence(model, B):
    # sequences of 0 to 3 tokens, empty ones in front, between and at the end
    lens = np.random.default_rng(B).integers(0, 4, size=B)
    if B > 2:
        lens[0] = lens[-1] = 0
    lens[B // 2] = 5
    pos = np.concatenate([np.arange(n) for n in lens])
    run, call = forward(model, lens)
    got = call()
    assert run.status() == 0
    run2, call2 = forward(model, lens, pos)
    assert torch.equal(got, call2()) and run2.status() == 0


@pytest.mark.parametrize("B,at", [(1, 0), (1025, 1024), (8200, 8199), (65535, 40000), (65535, 65534)])
def test_one_sequence_too_long_is_reported_wherever_it_is(model, B, at):
    lens = np.ones(B, dtype=np.int64)
    lens[at] = 3
    run, call = forward(model, lens, max_seqlen=2)
    call()
    assert run.status() == -6
    run, call = forward(model, lens)
    call()
    assert run.status() == 0


def test_checking_many_sequences_takes_little_time():
    # 64 tokens in 65000 sequences, all but the first of them empty, against the same 64 tokens alone; fp32, whose attention has
    # no work per sequence.  8 us more; 23 with a check whose loads wait for each other and a search by halves.
    cfg = synth.ModelConfig("many32", 1, 64, 1, 1, 16, 32, 512, "f32", max_pos=512)
    model = harness.upload_model(synth.SynthWeights(cfg, 5))

    def median_us(lens):
        run, call = forward(model, lens)
        out = call()
        times = []
        for _ in range(31):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                call(out)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 250.0)
        assert run.status() == 0
        return float(np.median(times))
    few = median_us([64])
    many = median_us([64] + [0] * 64999)
    model.close()
    print(f"1 sequence {few:.1f} us, 65000 sequences {many:.1f} us")
    assert many - few < 16.0
